// Forward kernels of one time step (HIP, gfx950).
//
// Storage. The state arrays hold fluid nodes only, indexed by fluid id (the rank of the node
// among fluid nodes in node order, so rows stay contiguous); thread t of a launch is fluid node t
// and writes its own slot, which makes every store a full coalesced line. Pulls find the id of
// the source node through a map of fluid bits and counts (IdWord). The small per-node fields
// (rho^N, the info word) stay dense, because the stencils also read them at solid nodes.
//
// State representation. Under Latva-Kokko recolouring of the colour-blind post-collision
// populations (eq. operator_recoloring) followed by the proportional wall-reaction transfer,
// the two colours' post-collision populations at a node are always
//     f^r_i = a f^m_i + (w_i/|c_i|) c_i . v,     f^p_i = b f^m_i - (w_i/|c_i|) c_i . v,
// with a = (1 - phi) rho^r / rho^m, b = 1 - a and v = (1 - phi) beta (rho^r rho^p / rho^m) n*. The
// state is therefore stored exactly as the 19 colour-blind populations f^m (storage precision),
// the four per-node scalars (a or b, v) (arithmetic precision) and, with the species, 7
// populations g: 30 values per node instead of 45. Pulling f^r_i from node x - c_i reads f^m_i
// and the scalars there.
//
// Near-pure phases. Where one colour is a trace (gas nucleating at a wall, a liquid film inside
// a bubble), storing a next to 1 or rho^N next to +-1 would round the trace colour to the
// absolute precision of the arithmetic type (6e-8 in FP32), and the interface normal, which
// divides by a gradient that may be as small as 1e-6, would be noise. Both are therefore kept
// in a minority form (pack_frac, rn_diff below): the smaller member of each pair (a, b) and
// ((1 + rho^N)/2, (1 - rho^N)/2) is stored at full relative precision, the sign bit telling
// which one it is. Colour densities and gradients of rho^N are formed from those directly.
//
// Layout: structure of arrays, one plane per population, planes a padded stride ps (at least the
// number of fluid nodes) apart, fluid ids in node order (x fastest); the colour scalars (a, v) as
// one 4-vector per fluid node. Two state buffers are used alternately (pull from one, write the
// other), so no kernel reads what another thread of the same launch writes.
//
// One step is four launches (each one thread per node; one, collide, where sigma = beta = 0):
//   colour   pull f^m, a, v -> rho^N at fluid nodes             (eqs. moments_components, color_function)
//   extrap   rho^N into solid nodes next to fluid               (eq. color_lattice_weighted_average)
//   normal   isotropic gradient, unit normal, Akai realignment   (eqs. finite_difference_scheme,
//                                                                 color_gradient_normal, realigned_normal_vectors)
//   collide  pull, curvature, forcing, central-moment collision, recolouring, reaction,
//            species, store, FP64 reductions                     (remaining equations)
// The 3-hop dependency rho^N -> n -> curvature between neighbours is what forces the split.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "lattice.hpp"
#include "precision.hpp"

namespace lbm {

constexpr int kBlock = 256;
constexpr int kXcd = 8;  // MI355X: 8 XCDs; workgroups are dealt round-robin across them

// Per-node vectors (colour scalars e, v; realigned normal; wetting data) are stored together so that
// one load brings all components: a gather's cost follows the cache lines it touches, so loading a
// subset of them costs about as much as all. The realigned normals, which the curvature gathers
// without |G|, are packed 3-vectors for the same reason: a wave's row of them covers six or
// seven cache lines, of 4-vectors eight or nine (512x512x128 collide: FP32 1081 -> 1059 us,
// FP16 878 -> 837 us).
template <class R> struct V4;
template <> struct V4<float> { using T = float4; };
template <> struct V4<double> { using T = double4; };
template <class R> struct V2;
template <> struct V2<float> { using T = float2; };
template <> struct V2<double> { using T = double2; };

// Element i of an array: with a 32-bit index type as a 32-bit byte offset from the (wave-uniform)
// base, which the caller knows to suffice; else with a 64-bit address.
template <class Off, class T>
__device__ inline T ldx(const T* base, Off i) {
  if constexpr (sizeof(Off) == 4)
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + uint32_t(i * uint32_t(sizeof(T))));
  else
    return base[i];
}
template <class Off, class T>
__device__ inline T& refx(T* base, Off i) {
  if constexpr (sizeof(Off) == 4)
    return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + uint32_t(i * uint32_t(sizeof(T))));
  else
    return base[i];
}
// Store of a value that no kernel reads before the caches have turned over (STREAM: nontemporal, so
// that it does not displace what they hold) or that one soon does.
template <bool STREAM, class T>
__device__ inline void put(T& dst, const T& v) {
  if constexpr (!STREAM) {
    dst = v;
  } else if constexpr (sizeof(T) == 2) {
    __builtin_nontemporal_store(__builtin_bit_cast(uint16_t, v), reinterpret_cast<uint16_t*>(&dst));
  } else if constexpr (sizeof(T) == 4) {
    __builtin_nontemporal_store(__builtin_bit_cast(uint32_t, v), reinterpret_cast<uint32_t*>(&dst));
  } else {
    static_assert(sizeof(T) == 8, "2, 4 or 8 bytes");
    __builtin_nontemporal_store(__builtin_bit_cast(uint64_t, v), reinterpret_cast<uint64_t*>(&dst));
  }
}
// Round one arm of a branch between such stores: without it the compiler merges the two arms into
// ordinary stores.
__device__ inline void keep_apart() { asm volatile("" ::: "memory"); }
template <class R>
struct Vec3 {
  R x, y, z;
};
// Element n of packed 3-vectors (the byte offset by shifts: a 32-bit product has a quarter of the rate).
template <class Off, class R>
__device__ inline Vec3<R>& ref3(R* p, Off n) {
  return *reinterpret_cast<Vec3<R>*>(&refx<Off>(p, Off((n << 1) + n)));
}
template <class Off, class R>
__device__ inline Vec3<R> ld3(const R* p, Off n) {
  return ref3<Off>(const_cast<R*>(p), n);
}
template <class Off, class R>
__device__ inline typename V4<R>::T ld4(const R* p, Off n) {
  return ldx<Off>(reinterpret_cast<const typename V4<R>::T*>(p), n);
}
template <class Off, class R>
__device__ inline void st4(R* p, Off n, R x, R y, R z, R w) {
  typename V4<R>::T v;
  v.x = x; v.y = y; v.z = z; v.w = w;
  refx<Off>(reinterpret_cast<typename V4<R>::T*>(p), n) = v;
}
template <class Off, class R>
__device__ inline void st4_stream(R* p, Off n, R x, R y, R z, R w) {
  typedef R V __attribute__((ext_vector_type(4)));
  const V v = {x, y, z, w};
  __builtin_nontemporal_store(v, reinterpret_cast<V*>(&refx<Off>(reinterpret_cast<typename V4<R>::T*>(p), n)));
}

// Uses all four components of a loaded vector. A load of which only some components are used is
// otherwise split, and a gather costs by the instruction and its cache lines, not by the words.
__device__ inline void use_whole(const float4& v) { asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w)); }
__device__ inline void use_whole(const double4& v) { asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w)); }

template <class T>
__device__ inline void use_whole(const T avs[18], const T edge[5]) {
#pragma unroll
  for (int i = 0; i < 18; ++i)
    if (D3Q19::cx[i] == 0) use_whole(avs[i]);
#pragma unroll
  for (int r = 0; r < 5; ++r) use_whole(edge[r]);
}

// a b rounded, never fused into a following sum.
template <class R>
__device__ inline R rounded_product(R a, R b) {
#pragma clang fp contract(off)
  return a * b;
}

// A pair of colour fractions (a, b), a + b = 1, stored as one number that holds the smaller one
// to full relative precision: e = -|b| (sign bit set) when 0 <= b <= a or a < 0, else e = |a|.
// So e = -0 is the pure reactant (red) state and e = +0 the pure product (blue) state; values
// outside [0, 1] (a colour density that rounded below zero) keep their sign consistently.
template <class R>
__device__ inline R pack_frac(R a, R b) {
  const bool minor_b = (b <= a && b >= R(0)) || a < R(0);
  return minor_b ? -fabs(b) : fabs(a);
}
template <class R>
__device__ inline void unpack_frac(R e, R& a, R& b) {
  const R minor = fabs(e), major = R(1) - minor;
  a = signbit(e) ? major : minor;
  b = signbit(e) ? minor : major;
}
// rho^N = a - b is stored as q = rho^N - s with s = +1 if the sign bit of q is set (product
// colour in the minority, q = -2b) and s = -1 otherwise (q = 2a).
template <class R>
__device__ inline R rn_side(R q) { return signbit(q) ? R(1) : R(-1); }
template <class R>
__device__ inline R rn_value(R q) { return q + rn_side(q); }
// rho^N(x) - rho^N(y) without the cancellation of two values next to +-1.
template <class R>
__device__ inline R rn_diff(R qx, R qy) { return (qx - qy) + (rn_side(qx) - rn_side(qy)); }
// q from the colour densities (rm = rho^r + rho^p up to rounding).
template <class R>
__device__ inline R rn_pack(R rr, R rp, R irm) { return R(2) * pack_frac(rr * irm, rp * irm); }
// rho^r and rho^p at a node from q and rho^m, the minority one directly.
template <class R>
__device__ inline void rn_densities(R q, R rm, R& rr, R& rp) {
  if (signbit(q)) {
    rp = R(-0.5) * q * rm;
    rr = rm - rp;
  } else {
    rr = R(0.5) * q * rm;
    rp = rm - rr;
  }
}

// Maps the hardware workgroup id to a logical tile so that each XCD (with its own L2) works on
// one contiguous slab of the lattice; neighbouring rows then share that XCD's L2.
// gridDim.x is always a multiple of kXcd.
// skip: leading workgroups without a tile (a multiple of kXcd).
__device__ inline int logical_block(int skip = 0) {
  const int per_xcd = (gridDim.x - skip) / kXcd, b = blockIdx.x - skip;
  return (b % kXcd) * per_xcd + b / kXcd;
}
// The same with runs of kRun workgroups dealt to the XCDs in turn (RUNS, large lattices; a workgroup is a tile, half
// a tile in FP64's colour pass): all XCDs
// then work on one window of the lattice that moves through it, instead of on eight far apart, and what
// two of them need is still in the last-level cache. Measured against the slabs: 512 x 512 x 128 FP32 colour
// 568 -> 560 us, extrap 81 -> 79, normal 205 -> 190; 256^3 FP16 normal 104 -> 98, colour 235 -> 234; runs of 8
// to 64 tiles differ by 1%, single tiles lose (colour 593). The collide pass, which streams more than it
// shares, gains nothing (FP16 811 -> 817). Workgroups past the last whole round keep their index.
constexpr int kRun = 64;
template <bool RUNS>
__device__ inline int run_block(int skip = 0) {
  if (!RUNS) return logical_block(skip);
  const int b = blockIdx.x - skip;
  if (b >= int(gridDim.x - skip) / (kXcd * kRun) * (kXcd * kRun)) return b;
  const int k = b / kXcd;
  return k / kRun * (kXcd * kRun) + b % kXcd * kRun + k % kRun;
}

// The tile of kBlock consecutive fluid ids that this workgroup processes: its XCD-aware launch
// index, through the context's tile order when there is one (on large lattices the tiles are
// launched in y-bands swept through z, so that tiles whose nodes neighbour each other across
// planes are in flight on the same XCD and share its L2).
template <class SA>
__device__ inline int fluid_tile(const SA& A) {
  const int lb = logical_block();
  return A.order ? A.order[lb] : lb;
}
// The fluid id of this thread where a tile is shared by kBlock / THREADS workgroups.
template <int THREADS, bool RUNS, class SA>
__device__ inline uint32_t split_tile_id(const SA& A, int skip) {
  constexpr int kParts = kBlock / THREADS;
  const int lb = run_block<RUNS>(skip), tile = lb / kParts, part = lb % kParts;
  return uint32_t(A.order ? A.order[tile] : tile) * kBlock + uint32_t(part) * THREADS + threadIdx.x;
}

// Division by a runtime constant d for 0 <= n < 2^31: q = (umulhi(n, m) + n) >> s with
// s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1 (computed on the host).
struct FastDiv {
  uint32_t d, m, s;
  __device__ inline uint32_t div(uint32_t n) const { return (__umulhi(n, m) + n) >> s; }
};

struct Geom {
  int nx, ny, nz;
  FastDiv fx, fy;
};

// All ones where bit i of w is set, else zero, and selects by such masks. The masks stay in vector
// registers and each select is one v_bfi: a lane mask in scalar registers costs a compare per use
// (18 link bits do not stay resident) and two wait states between the compare and the select. The
// instruction is written out because the compiler turns the builtin back into compare and select.
__device__ inline uint32_t bit_mask(uint32_t w, int i) {
  uint32_t m = 0u - ((w >> i) & 1u);
  if (__builtin_constant_p(i)) asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(w), "n"(i));
  return m;
}
__device__ inline uint32_t blend(uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); }
__device__ inline float blend(uint32_t m, float a, float b) {
  return __uint_as_float(blend(m, __float_as_uint(a), __float_as_uint(b)));
}
__device__ inline double blend(uint32_t m, double a, double b) {
  const uint64_t x = uint64_t(__double_as_longlong(a)), y = uint64_t(__double_as_longlong(b));
  return __longlong_as_double((long long)((uint64_t(blend(m, uint32_t(x >> 32), uint32_t(y >> 32))) << 32) |
                                          blend(m, uint32_t(x), uint32_t(y))));
}
__device__ inline float2 blend(uint32_t m, const float2& a, const float2& b) {
  return make_float2(blend(m, a.x, b.x), blend(m, a.y, b.y));
}
__device__ inline double2 blend(uint32_t m, const double2& a, const double2& b) {
  return make_double2(blend(m, a.x, b.x), blend(m, a.y, b.y));
}
template <class R>
__device__ inline Vec3<R> blend(uint32_t m, const Vec3<R>& a, const Vec3<R>& b) {
  return {blend(m, a.x, b.x), blend(m, a.y, b.y), blend(m, a.z, b.z)};
}
__device__ inline float4 blend(uint32_t m, const float4& a, const float4& b) {
  return make_float4(blend(m, a.x, b.x), blend(m, a.y, b.y), blend(m, a.z, b.z), blend(m, a.w, b.w));
}
__device__ inline double4 blend(uint32_t m, const double4& a, const double4& b) {
  return make_double4(blend(m, a.x, b.x), blend(m, a.y, b.y), blend(m, a.z, b.z), blend(m, a.w, b.w));
}

// A masked load leaves its destination unset in the lanes without it, and a blend that drops such a value is
// still undefined to the compiler, which may then drop the blend: the destination is given a value first.
// Zero, or where this is faster, whichever value the register holds (no instruction; the number keeps the
// compiler from merging several into one, and a volatile statement, which needs none, would hold the
// instructions round it in place). One-kernel step, FP64 128^3: 98.8 us with the id words and the row edges
// unset, 98.9 with this for the words and zeros for the edges, 99.2 with zeros, 100.1 with this for both.
template <class T>
__device__ inline void any_value(T& v, int number) {
  v = T(0);
  if (__builtin_constant_p(number)) asm("; %1" : "=v"(v) : "n"(number));  // (zero in builds that do not fold it)
}

// Entry of a launch list.
struct ListNode {
  int node;
  uint32_t info;  // its info word, with the face bits
};

// Periodic neighbour offsets of one node.
struct Nbr {
  int n;
  int dxm, dxp, dym, dyp, dzm, dzp;
  __device__ inline int at(int cx, int cy, int cz) const {
    return n + (cx > 0 ? dxp : (cx < 0 ? dxm : 0)) + (cy > 0 ? dyp : (cy < 0 ? dym : 0)) +
           (cz > 0 ? dzp : (cz < 0 ? dzm : 0));
  }
};

// From the face bits: the division of n by the lattice sizes takes five products at a quarter of the
// rate, a tenth of the colour pass's instruction time.
__device__ inline Nbr make_nbr(int n, uint32_t inf, const Geom& g) {
  const int nx = g.nx, nxy = g.nx * g.ny, N = nxy * g.nz;
  auto face = [&](int k) { return int(bit_mask(inf, kFaceShift + k)); };
  Nbr b;
  b.n = n;
  b.dxm = (face(0) & nx) - 1;
  b.dxp = 1 - (face(1) & nx);
  b.dym = (face(2) & nxy) - nx;
  b.dyp = nx - (face(3) & nxy);
  b.dzm = (face(4) & N) - nxy;
  b.dzp = nxy - (face(5) & N);
  return b;
}

// Direction with no x component and the same y and z components as direction i (-1 for the
// x axis, whose counterpart is the rest position).
constexpr int yz_partner(int i) {
  for (int j = 0; j < 18; ++j)
    if (D3Q19::cx[j] == 0 && D3Q19::cy[j] == D3Q19::cy[i] && D3Q19::cz[j] == D3Q19::cz[i]) return j;
  return -1;
}

// Map from nodes to fluid ids. Word w covers the nodes n = 32 w .. 32 w + 31: the bits of the fluid
// ones, and the number of fluid nodes before the first of them in dense order. The number of fluid
// nodes before any node, fluid or solid, is then a bit count away, and at a fluid node that is its
// id. Against a dense map (4 bytes per node) it takes a sixteenth of the bytes, and the lookups of a
// wave, whose nodes span about 64 / porosity of a row, touch one or two cache lines per row instead
// of four. Measured with the dense map: 512 x 512 x 128 porous, FP32, colour 604 -> 580 us and
// collide 1123 -> 1084 us; at 128^3, which stays in the last-level cache, the same time.
struct IdWord {
  uint32_t fluid, before;
};
__device__ inline uint32_t fluid_before(IdWord w, uint32_t n) { return __popc(w.fluid & ((1u << (n & 31u)) - 1u)) + w.before; }
__device__ inline bool is_fluid(IdWord w, uint32_t n) { return (w.fluid >> (n & 31u)) & 1u; }
__device__ inline uint32_t fluid_id(const IdWord* ids, int n) { return fluid_before(ids[n >> 5], uint32_t(n)); }

// Fluid ids of the 18 pull sources x - c_i of fluid node t, the node's own id where the source is
// solid. With the count r of fluid nodes before the row centre x - (0, c_iy, c_iz), a fluid source
// one node before it on the row has id r - 1 and one after it r + 1 (r where the centre is solid),
// so eight lookups give all 18 ids; only a lane at a periodic x face looks up the five sources
// across the face. All lookups are issued before any id is formed.
template <class Off>
__device__ inline void pull_sources(const IdWord* ids, const Nbr& nb, uint32_t t, uint32_t inf, uint32_t sid[18]) {
  using D = D3Q19;
  uint32_t centre[18];
  IdWord w[18];
#pragma unroll
  for (int i = 0; i < 18; ++i)
    if (D::cx[i] == 0) {
      centre[i] = uint32_t(nb.at(0, -D::cy[i], -D::cz[i]));
      w[i] = ldx<Off>(ids, centre[i] >> 5);
    }
  const uint32_t low = bit_mask(inf, kFaceShift), high = bit_mask(inf, kFaceShift + 1);
  // the source across the x face on the node's own row (1) and the rows of directions 2..5
  IdWord aw[6];
  const uint32_t dx = uint32_t(blend(low, uint32_t(nb.dxm), uint32_t(nb.dxp)));  // a row of one node has both, the same node
  centre[1] = uint32_t(nb.n);
#pragma unroll
  for (int i = 1; i < 6; ++i) {
    any_value(aw[i].fluid, 2 * i);
    any_value(aw[i].before, 2 * i + 1);
  }
  if (low | high) {
#pragma unroll
    for (int i = 1; i < 6; ++i) aw[i] = ldx<Off>(ids, (centre[i] + dx) >> 5);
  }
  uint32_t r[18], across[6];
#pragma unroll
  for (int i = 1; i < 6; ++i) across[i] = fluid_before(aw[i], centre[i] + dx);
#pragma unroll
  for (int i = 0; i < 18; ++i)
    if (D::cx[i] == 0) r[i] = fluid_before(w[i], centre[i]);
#pragma unroll
  for (int i = 0; i < 18; ++i) {
    const int m = yz_partner(i);
    uint32_t id;
    if (D::cx[i] == 0) {
      id = r[i];
    } else if (D::cx[i] > 0) {
      id = blend(low, across[m < 0 ? 1 : m], (m < 0 ? t : r[m]) - 1u);
    } else {
      id = blend(high, across[m < 0 ? 1 : m], m < 0 ? t + 1u : r[m] + 1u + bit_mask(inf, m));
    }
    sid[i] = blend(bit_mask(inf, i), t, id);
  }
}

// Cross-lane moves within the 64-wide wave (DPP wave shifts, one VALU move per 32-bit word): the
// value that lane l - 1 (from_below) or lane l + 1 (from_above) holds in the same register. The end
// lanes of the wave receive zero; callers use the result only where the neighbouring lane is
// active and holds the wanted node.
__device__ inline int lane_from_below(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ inline int lane_from_above(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
template <int DIR>
__device__ inline float lane_move(float v) {
  const int b = __float_as_int(v);
  return __int_as_float(DIR < 0 ? lane_from_below(b) : lane_from_above(b));
}
template <int DIR>
__device__ inline double lane_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = int(uint32_t(b)), hi = int(uint32_t(uint64_t(b) >> 32));
  const int mlo = DIR < 0 ? lane_from_below(lo) : lane_from_above(lo);
  const int mhi = DIR < 0 ? lane_from_below(hi) : lane_from_above(hi);
  return __longlong_as_double((long long)((uint64_t(uint32_t(mhi)) << 32) | uint32_t(mlo)));
}
template <int DIR>
__device__ inline float2 lane_move(const float2& v) {
  return make_float2(lane_move<DIR>(v.x), lane_move<DIR>(v.y));
}
template <int DIR>
__device__ inline double2 lane_move(const double2& v) {
  return make_double2(lane_move<DIR>(v.x), lane_move<DIR>(v.y));
}
template <int DIR, class R>
__device__ inline Vec3<R> lane_move(const Vec3<R>& v) {
  return {lane_move<DIR>(v.x), lane_move<DIR>(v.y), lane_move<DIR>(v.z)};
}
template <int DIR>
__device__ inline float4 lane_move(const float4& v) {
  return make_float4(lane_move<DIR>(v.x), lane_move<DIR>(v.y), lane_move<DIR>(v.z), lane_move<DIR>(v.w));
}
template <int DIR>
__device__ inline double4 lane_move(const double4& v) {
  return make_double4(lane_move<DIR>(v.x), lane_move<DIR>(v.y), lane_move<DIR>(v.z), lane_move<DIR>(v.w));
}

// Values of a per-node quantity at the 18 neighbours x - c_i of fluid node x (out[i]), fetched with
// one gather per row. The sources x - c_i with c_ix != 0 lie on the row of the source
// x - (0, c_iy, c_iz) of the partner direction, one node along x; when the node's own neighbour
// x - c_ix along the row is fluid, it is the next fluid id and lane l - c_ix of the same wave holds
// it, and that lane's partner value is exactly the one wanted. Those values are moved across lanes
// instead of gathered, so each row triple costs one gather for all lanes. The lanes that cannot be
// served so (wave ends, periodic wrap, a solid neighbour along x) lack one of the row's two shifted
// sources: the first node of a run of fluid nodes the one before it, the last node the one after it.
// Both kinds share one masked gather per row, each lane with the index of the source it lacks; the
// few lanes that lack both (runs of a single node; 6% of the waves of the 512^3 mask, 16% of the
// 128^3 one have such a lane) fetch the second one in a branch of their own.
// idx(i): the index of the source of direction i; ld(k): the value at index k. own is the node's own
// value (the source of the x-shifted directions of the node's own row). SOLID_OWN: where x - c_i is
// solid the node's own value stands in (state vectors, whose solid sources are bounce-back);
// otherwise every neighbour has a value of its own (rho^N, extrapolated into solids). need(i): false
// (a constant) for a direction whose value is neither used nor the centre of one that is.
// Every 64 consecutive threads of a launch hold consecutive fluid ids.
// row_gather issues the gathers; row_resolve waits for them and moves the values across lanes, so a
// caller can put its other loads in flight between the two.
constexpr int kRowPlus[5] = {0, 6, 7, 8, 9}, kRowMinus[5] = {1, 10, 11, 12, 13};  // directions (+1, r), (-1, r) of row r

struct RowLanes {
  bool below, above;  // lane l - 1 holds node x - 1 of this row (direction 0 pulls from x - 1), lane l + 1 node x + 1
};
__device__ inline RowLanes row_lanes(uint32_t inf) {
  const int lane = __lane_id();
  return {!(inf & (1u | (1u << kFaceShift))) && lane > 0, !(inf & (2u | (2u << kFaceShift))) && lane < 63};
}

template <bool SOLID_OWN, class T, class Index, class Load, class Need>
__device__ inline void row_gather(const RowLanes& lanes, uint32_t inf, Index idx, Load ld, Need need, T out[18], T edge[5]) {
  using D = D3Q19;
  const bool below = lanes.below, above = lanes.above;
  const uint32_t belowm = below ? ~0u : 0u, abovem = above ? ~0u : 0u;
#pragma unroll
  for (int r = 0; r < 5; ++r) edge[r] = T{};
#pragma unroll
  for (int i = 0; i < 18; ++i)
    if (D::cx[i] == 0 && need(i)) out[i] = ld(idx(i));
#pragma unroll
  for (int r = 0; r < 5; ++r) {
    const int ip = kRowPlus[r], im = kRowMinus[r];
    if (!need(ip)) continue;
    const uint32_t lack_p = SOLID_OWN ? ~(belowm | bit_mask(inf, ip)) : ~belowm;
    const uint32_t lack_m = SOLID_OWN ? ~(abovem | bit_mask(inf, im)) : ~abovem;
    if (lack_p | lack_m) edge[r] = ld(blend(lack_p, idx(ip), idx(im)));
  }
}

template <bool SOLID_OWN, class T, class Index, class Load, class Need>
__device__ inline void row_resolve(const RowLanes& lanes, uint32_t inf, const T& own, Index idx, Load ld, Need need,
                                   T out[18], const T edge[5]) {
  const bool below = lanes.below, above = lanes.above;
  const uint32_t belowm = below ? ~0u : 0u, abovem = above ? ~0u : 0u;
#pragma unroll
  for (int r = 0; r < 5; ++r) {
    const int ip = kRowPlus[r], im = kRowMinus[r];
    if (!need(ip)) continue;
    const int m = yz_partner(ip);
    const T base = (m < 0) ? own : out[m];
    out[ip] = blend(belowm, lane_move<-1>(base), edge[r]);
    out[im] = blend(abovem, lane_move<+1>(base), edge[r]);
  }
  if (!below && !above) {
#pragma unroll
    for (int r = 0; r < 5; ++r)
      if (need(kRowPlus[r])) out[kRowMinus[r]] = ld(idx(kRowMinus[r]));
  }
  if (SOLID_OWN) {
#pragma unroll
    for (int r = 0; r < 5; ++r) {
      const int ip = kRowPlus[r], im = kRowMinus[r];
      if (!need(ip)) continue;
      out[ip] = blend(bit_mask(inf, ip), own, out[ip]);
      out[im] = blend(bit_mask(inf, im), own, out[im]);
    }
  }
}

template <bool SOLID_OWN, class T, class Index, class Load, class Need>
__device__ inline void row_shared(uint32_t inf, const T& own, Index idx, Load ld, Need need, T out[18]) {
  const RowLanes lanes = row_lanes(inf);
  T edge[5];
  row_gather<SOLID_OWN>(lanes, inf, idx, ld, need, out, edge);
  row_resolve<SOLID_OWN>(lanes, inf, own, idx, ld, need, out, edge);
}

template <int P>
struct StepArgs {
  using S = typename Prec<P>::S;
  using R = typename Prec<P>::R;
  using Off = typename Prec<P>::Off;
  int nx, ny, nz, N;
  size_t ps;              // plane stride of the state and adjoint planes (>= fluid nodes)
  Geom geo;
  const ListNode* fluid;  // the fluid nodes, in increasing order
  int nfluid;
  const ListNode* ext;    // the solid nodes whose colour is extrapolated
  int next;
  const IdWord* ids;      // map from nodes to fluid ids (index into the state arrays)
  const int* order;       // optional launch order of the fluid-list tiles (null: list order)
  const uint32_t* info;
  int stream_vectors;  // nontemporal stores of the per-node vectors that one pass leaves to the next
  // state in (pull source) and out
  const S* fin;  // 19 planes f^m
  const R* ain;  // per node 4-vector (e, vx, vy, vz), e = pack_frac(a, b)
  const S* gin;  // 7 planes species
  const R* cin;  // 2-byte storages: the species total of each node (deviation reference of gin)
  S* fout;
  R* aout;
  S* gout;
  R* cout;
  R* rhoN;       // 1 plane, rho^N in the form of rn_value
  R* rm_out;     // optional: rho^m of each fluid node (adjoint recompute)
  R* nst;        // per fluid id packed 3-vector n*
  R* glen;       // per fluid id |grad rho^N|
  R* nraw;       // optional: per fluid id, the unit normal before the wetting realignment at
                 // wetting nodes (kept for the adjoint; elsewhere it equals n*)
  const R* wet;  // per fluid id 4-vector (n_s, cos(theta))
  double* partials;  // per-workgroup sums of the step (null: none wanted)
  // Deferred final reduction of the previous step, done by the step's first pass (null: none)
  const double* red_in;
  int red_n;
  double* red_out;
  R relax;           // 1 - 1/tau
  R inv_tau_c;
  R sigma, beta, xi, c_in, eps;
  R acc[2][3];
  R scale, inv_scale;
  R gscale, inv_gscale;
  int species;
  // moments mode outputs (may be null)
  R* m_rr;
  R* m_rp;
  R* m_rn;
  R* m_u;
  R* m_c;
};

// Species storage. FP32 and FP64 hold the populations g_q themselves. The 2-byte storages hold
// each node's post-collision species total C (arithmetic type, plane cin/cout) and the
// populations as deviations (g_q - w_q C) 2^k from the equilibrium at rest of that total: those
// are small (advection and non-equilibrium parts only) wherever C lies in [0, 1], so the 11 or 8
// significant bits of the storage apply to them and not to C itself. Population q of the node with
// fluid id src:
template <int P>
__device__ inline typename Prec<P>::R species_value(const StepArgs<P>& A, int q, typename Prec<P>::Off src, typename Prec<P>::S s) {
  using R = typename Prec<P>::R;
  const R w = R(D3Q7::w(q));
  return Prec<P>::ld(s, Prec<P>::deviations ? w * ldx<typename Prec<P>::Off>(A.cin, src) : w, A.inv_gscale);
}
template <int P>
__device__ inline typename Prec<P>::R ld_species(const StepArgs<P>& A, int q, typename Prec<P>::Off src) {
  return species_value(A, q, src, ldx<typename Prec<P>::Off>(A.gin + size_t(q) * A.ps, src));
}

// The stored population that a pull along direction i reads from plane i at src, or from the plane
// of the opposite direction where bit i of inf is set (bounce-back; src is then the node itself).
// The two planes share one uniform base, that of the lower one, and the select adds their distance.
template <class Off, class S>
__device__ inline S& ref_pull(S* planes, size_t ps, int i, int opp, uint32_t src, uint32_t inf) {
  const int lo = i < opp ? i : opp, dist = i < opp ? opp - i : i - opp;
  const uint32_t upper = bit_mask(i < opp ? inf : ~inf, i);
  return refx<Off>(planes + size_t(lo) * ps, Off(src) + (Off(int64_t(int32_t(upper))) & Off(size_t(dist) * ps)));
}
template <class Off, class S>
__device__ inline S ld_pull(const S* planes, size_t ps, int i, int opp, uint32_t src, uint32_t inf) {
  return ref_pull<Off>(const_cast<S*>(planes), ps, i, opp, src, inf);
}

// Pull of fluid node t with halfway bounce-back: f^m_i from S_t at x - c_i, or S_t,opp(i) at x
// where x - c_i is solid (sid: the sources' fluid ids, t for bounce-back), as stored; and likewise the
// species (the outflow plane takes its own S_1: zero gradient).
template <int P>
__device__ inline void ld_populations(const StepArgs<P>& A, uint32_t t, uint32_t inf, const uint32_t sid[18],
                                      typename Prec<P>::S s[19]) {
  using Off = typename Prec<P>::Off;
#pragma unroll
  for (int i = 0; i < 18; ++i) s[i] = ld_pull<Off>(A.fin, A.ps, i, D3Q19::opp[i], sid[i], inf);
  s[18] = ldx<Off>(A.fin + 18 * A.ps, t);
}
template <int P>
__device__ inline void pull_species(const StepArgs<P>& A, uint32_t t, uint32_t inf, const uint32_t sid[18],
                                    typename Prec<P>::R g[7]) {
  using Off = typename Prec<P>::Off;
#pragma unroll
  for (int i = 0; i < 7; ++i) g[i] = 0;
  if (A.species) {
    const bool outlet = inf & kOutlet;  // zero-gradient outflow: the node's own S_1
    const uint32_t ginf = outlet ? inf & ~2u : inf;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const uint32_t src = (i == 1 && outlet) ? t : sid[i];
      g[i] = species_value(A, i, src, ld_pull<Off>(A.gin, A.ps, i, D3Q7::opp[i], src, ginf));
    }
    g[6] = ld_species(A, 6, t);
  }
}

// The wave's sums of four values per lane: lane l receives the sum of value l / 16. Two exchanges of
// wave halves and rows (v_permlane32_swap, v_permlane16_swap: each leaves two half-summed values
// in one register) and four rotations within rows of 16, 21 vector instructions and no LDS; five
// separate butterflies took 60 LDS permutes and 30 additions, a third of the collide pass's tail.
__device__ inline double from_words(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
}
__device__ inline void to_words(double v, uint32_t& lo, uint32_t& hi) {
  const uint64_t b = uint64_t(__double_as_longlong(v));
  lo = uint32_t(b);
  hi = uint32_t(b >> 32);
}
// (a over both wave halves) in the lower lanes, (b over both) in the upper ones
__device__ inline double fold_halves(double a, double b) {
  uint32_t al, ah, bl, bh;
  to_words(a, al, ah);
  to_words(b, bl, bh);
  const auto lo = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
  return from_words(lo[0], hi[0]) + from_words(lo[1], hi[1]);
}
// (a over row pairs) in the even rows of 16 lanes, (b over row pairs) in the odd ones
__device__ inline double fold_rows(double a, double b) {
  uint32_t al, ah, bl, bh;
  to_words(a, al, ah);
  to_words(b, bl, bh);
  const auto lo = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
  return from_words(lo[0], hi[0]) + from_words(lo[1], hi[1]);
}
template <int K>  // the value of the lane K before in the row, rotating (DPP row_ror)
__device__ inline double rotate_row(double v) {
  uint32_t lo, hi;
  to_words(v, lo, hi);
  return from_words(uint32_t(__builtin_amdgcn_update_dpp(0, int(lo), 0x120 + K, 0xf, 0xf, true)),
                    uint32_t(__builtin_amdgcn_update_dpp(0, int(hi), 0x120 + K, 0xf, 0xf, true)));
}
__device__ inline double wave_sums(double s0, double s1, double s2, double s3) {
  double v = fold_rows(fold_halves(s0, s2), fold_halves(s1, s3));
  v += rotate_row<8>(v);
  v += rotate_row<4>(v);
  v += rotate_row<2>(v);
  v += rotate_row<1>(v);
  return v;
}

// Sum of the per-workgroup partials (5 planes of nparts) by one workgroup, in a fixed order: strided
// sums of kBlock slots, then each 64 slots' sums, then those in order. A workgroup of fewer threads
// takes the slots in turn, so a step's sums do not depend on where the reduction ran.
template <int THREADS>
__device__ inline void reduce_partials(const double* partials, int nparts, double* out) {
  __shared__ double red[kBlock / 64][5];
  const int lane = threadIdx.x & 63;
  for (int slot = threadIdx.x; slot < kBlock; slot += THREADS) {
    double t[5] = {0, 0, 0, 0, 0};
    int b = slot;
    for (; b + 3 * kBlock < nparts; b += 4 * kBlock) {
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const double* p = partials + size_t(j) * nparts;
        t[j] += ((p[b] + p[b + kBlock]) + (p[b + 2 * kBlock] + p[b + 3 * kBlock]));
      }
    }
    for (; b < nparts; b += kBlock) {
#pragma unroll
      for (int j = 0; j < 5; ++j) t[j] += partials[size_t(j) * nparts + b];
    }
    const double v = wave_sums(t[0], t[1], t[2], t[3]), v4 = wave_sums(t[4], 0.0, 0.0, 0.0);
    if (lane % 16 == 0) red[slot >> 6][lane / 16] = v;
    if (lane == 0) red[slot >> 6][4] = v4;
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    double sum = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) sum += red[w][threadIdx.x];
    out[threadIdx.x] = sum;
  }
}

// The sums of the last step of a chunk into its ring row, then rows 0 .. rows - 1 to host memory
// (pinned: the kernel's own stores spare the copy and its wait, 8 of the 46 us of a one-step call).
__global__ __launch_bounds__(kBlock) void k_finish_reduce(const double* partials, int nparts, double* ring, int rows,
                                                          double* host) {
  reduce_partials<kBlock>(partials, nparts, ring + 5 * (rows - 1));
  __syncthreads();
  if (host)
    for (int i = threadIdx.x; i < 5 * rows; i += kBlock) host[i] = ring[i];
}

// A step's first kernel is launched with kXcd workgroups more when it also finishes the previous step's
// sums (red_out): workgroup 0 does only that, the other seven return, so that no tile waits for the
// sums, and the rest keep their XCD. True if the workgroup has no tile.
template <int THREADS, class SA>
__device__ inline bool finish_previous(const SA& A) {
  if (!A.red_out || blockIdx.x >= kXcd) return false;
  if (blockIdx.x == 0) reduce_partials<THREADS>(A.red_in, A.red_n, A.red_out);
  return true;
}

// ---------------------------------------------------------------------------------------------
// colour: rho^N = (rho^r - rho^p)/rho^m from the pulled populations. Two dependent round trips (the
// id map, then every gather of the node: nine rows of colour scalars, the rows' edges and 19
// populations, all in flight together). Bound by the cache requests of its gathers, not by
// instructions or occupancy: with every source replaced by the node itself (the same loads, aligned)
// it takes 417 us on a 512 x 512 x 128 porous lattice (18.5M fluid nodes, FP32), as a plain read of
// its planes does, and with the real sources 576 us (118 B per node, 3.8 TB/s; 650 us before the
// id words, the merged row edges and the 32-bit offsets, 560 with the stores and the launch order of
// large lattices); 128^3 FP32 37.2 -> 34.8 us, FP64 84.8 -> 69.6 us (62 with half-size workgroups and
// nontemporal stores of the state). 94 VGPRs, five waves per SIMD; holding it to four costs 4%.
// ---------------------------------------------------------------------------------------------

// rho^N (rn_value form) and rho^m of a node from its pulled populations fm(i) and the colour scalars
// (e, v): own, and avs[i] of the node at x - c_i (of any node where that is solid and c_ix != 0; own
// where it is solid and c_ix = 0). Every pass that forms rho^N calls this.
template <class R, class Pop>
__device__ inline R colour_of(uint32_t inf, const typename V4<R>::T& own, const typename V4<R>::T avs[18], Pop fm, R& rm_out) {
  using D = D3Q19;
  // c_i . v, without the terms of zero components
  const auto along = [](int i, const typename V4<R>::T& av) {
    R s = 0;
    bool first = true;
    if (D::cx[i]) { s = D::cx[i] > 0 ? av.y : -av.y; first = false; }
    if (D::cy[i]) { const R w = D::cy[i] > 0 ? av.z : -av.z; s = first ? w : s + w; first = false; }
    if (D::cz[i]) { const R w = D::cz[i] > 0 ? av.w : -av.w; s = first ? w : s + w; }
    return s;
  };
  R rm = 0, rr = 0, rp = 0;
#pragma unroll
  for (int i = 0; i < 18; ++i) {
    const R f = fm(i);
    // where x - c_i is solid, the node's own population of direction opp(i) bounced back
    const uint32_t bb = bit_mask(inf, i);
    const R e = D::cx[i] ? blend(bb, own.x, avs[i].x) : avs[i].x;
    const R cv = blend(bb, along(D::opp[i], own), along(i, avs[i]));
    R a, b;
    unpack_frac(e, a, b);
    const R kv = rounded_product(R(D::w_over_len(i)), cv);
    rm += f;
    rr += a * f + kv;
    rp += b * f - kv;
  }
  const R f0 = fm(18);
  R a0, b0;
  unpack_frac(own.x, a0, b0);
  rm += f0;
  rr += rounded_product(a0, f0);
  rp += rounded_product(b0, f0);
  rm_out = rm;
  return rn_pack(rr, rp, R(1) / rm);
}

template <int P, int THREADS, bool LARGE>
__global__ __launch_bounds__(THREADS) void k_colour(StepArgs<P> A) {
  using R = typename Prec<P>::R;
  using D = D3Q19;
  using Off = typename Prec<P>::Off;
  if (finish_previous<THREADS>(A)) return;
  const uint32_t t = split_tile_id<THREADS, LARGE>(A, A.red_out ? kXcd : 0);
  if (t >= uint32_t(A.nfluid)) return;
  const ListNode ln = ldx<Off>(A.fluid, t);
  const int n = ln.node;
  const uint32_t inf = ln.info;
  const Nbr nb = make_nbr(n, inf, A.geo);
  uint32_t sid[18];
  pull_sources<Off>(A.ids, nb, t, inf, sid);
  const typename V4<R>::T own = ld4<Off>(A.ain, t);
  typename V4<R>::T avs[18], edge[5];  // (e, v) at the sources
  const RowLanes lanes = row_lanes(inf);
  const auto idx = [&](int i) { return sid[i]; };
  const auto ld = [&](uint32_t k) { return ld4<Off>(A.ain, k); };
  const auto all = [](int) { return true; };
  row_gather<true>(lanes, inf, idx, ld, all, avs, edge);
  typename Prec<P>::S s[19];
  ld_populations(A, t, inf, sid, s);
  __builtin_amdgcn_sched_barrier(0);  // every load of the node in flight before the first wait
  use_whole(avs, edge);
  row_resolve<false>(lanes, inf, own, idx, ld, all, avs, edge);
  R rm;
  const R q = colour_of<R>(inf, own, avs, [&](int i) { return Prec<P>::ld(s[i], R(D::w(i)), A.inv_scale); }, rm);
  refx<Off>(A.rhoN, uint32_t(n)) = q;
  if (A.rm_out) refx<Off>(A.rm_out, uint32_t(n)) = rm;
}

// ---------------------------------------------------------------------------------------------
// extrap: colour of solid nodes next to fluid, lattice-weighted average of fluid neighbours.
// ---------------------------------------------------------------------------------------------
template <int P, bool LARGE>
__global__ __launch_bounds__(kBlock) void k_extrap(StepArgs<P> A) {
  using R = typename Prec<P>::R;
  using D = D3Q19;
  using Off = typename Prec<P>::Off;
  const uint32_t t = uint32_t(run_block<LARGE>()) * kBlock + threadIdx.x;
  if (t >= uint32_t(A.next)) return;
  const ListNode ln = ldx<Off>(A.ext, t);
  const int n = ln.node;
  const uint32_t inf = ln.info;
  const Nbr nb = make_nbr(n, inf, A.geo);
  // All 18 loads are issued before any is used, so their latencies overlap; a direction without a
  // fluid neighbour loads nothing (its lanes are masked off, which spares the address units; reading
  // the node's own entry instead made the pass 11% slower at 128^3).
  R qv[18];
#pragma unroll
  for (int i = 0; i < 18; ++i) {
    qv[i] = R(0);
    if ((inf >> i) & 1u) qv[i] = ldx<Off>(A.rhoN, uint32_t(nb.at(D::cx[i], D::cy[i], D::cz[i])));
  }
  // Weighted sums of the offsets q and of the sides s separately; -0 as the start keeps the
  // sign of an all-(-0) sum.
  R nq = R(-0.0), ns = 0, den = 0;
#pragma unroll
  for (int i = 0; i < 18; ++i) {
    const bool use = (inf >> i) & 1u;
    nq = use ? nq + R(D::w(i)) * qv[i] : nq;
    ns = use ? ns + R(D::w(i)) * rn_side(qv[i]) : ns;
    den = use ? den + R(D::w(i)) : den;
  }
  if (ns == den || ns == -den) {
    refx<Off>(A.rhoN, uint32_t(n)) = nq / den;  // all neighbours on one side: the average keeps that side
  } else {
    const R v = (ns + nq) / den;
    refx<Off>(A.rhoN, uint32_t(n)) = R(2) * pack_frac(R(0.5) * (R(1) + v), R(0.5) * (R(1) - v));
  }
}

// ---------------------------------------------------------------------------------------------
// normal: G = 3 sum_i w_i c_i rho^N(x + c_i) as pair differences (a uniform field gives exactly
// zero), n = +G/|G| (the opposite of the sign printed in eq. color_gradient_normal: with +G the
// force, curvature, recolouring and wetting angle all act with the physical sign, theta measured
// through the reactant colour), and at wetting nodes the Akai realignment
// n* = n+ (n+ is always at least as close to n as n-: n+.n - n-.n = 2 sin(theta) sin(theta')).
// ---------------------------------------------------------------------------------------------
// The normal of one fluid node from the nine pair differences d_j = rho^N(x + c_p) - rho^N(x - c_p),
// p = half[j], of its neighbours' colour (rn_diff form): G, |G|, n = G/|G|, and at wetting nodes
// the Akai realignment with wv = (n_s, cos(theta)). raw: the unit normal before realignment, set
// (and raw_set true) at wetting nodes with |G| > eps. Every pass that forms a normal calls this.
template <class R>
__device__ inline void normal_from_pairs(const R d[9], uint32_t inf, const typename V4<R>::T& wv, R eps, R nv[3],
                                         R& len, R raw[3], bool& raw_set) {
  using D = D3Q19;
  R g[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const int p = D::half[j];
    const R c3w = R(3.0 * D::w(p));
    if (D::cx[p]) g[0] += c3w * R(D::cx[p]) * d[j];
    if (D::cy[p]) g[1] += c3w * R(D::cy[p]) * d[j];
    if (D::cz[p]) g[2] += c3w * R(D::cz[p]) * d[j];
  }
  len = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
  nv[0] = nv[1] = nv[2] = R(0);
  raw_set = false;
  if (len > eps) {
    const R il = R(1) / len;
    nv[0] = g[0] * il; nv[1] = g[1] * il; nv[2] = g[2] * il;
    if (inf & kWet) {
      raw[0] = nv[0]; raw[1] = nv[1]; raw[2] = nv[2];
      raw_set = true;
      const R sx = wv.x, sy = wv.y, sz = wv.z;
      if (sx * sx + sy * sy + sz * sz > R(0.5)) {
        const R ct = wv.w;
        const R st = sqrt(fmax(R(0), (R(1) - ct) * (R(1) + ct)));
        // cos and sin of theta' from the dot and cross products (accurate next to +-n_s).
        const R cp = sx * nv[0] + sy * nv[1] + sz * nv[2];
        const R q0 = nv[1] * sz - nv[2] * sy, q1 = nv[2] * sx - nv[0] * sz, q2 = nv[0] * sy - nv[1] * sx;
        const R sp = sqrt(q0 * q0 + q1 * q1 + q2 * q2);
        // n+ = cos(theta) n_s + sin(theta) t, t = (n - cos(theta') n_s)/sin(theta'): n rotated in
        // the plane of n and n_s to the angle theta. Within sin(theta') < 1e-2 of +-n_s that plane
        // is not defined by n (an interface parallel to the wall) and n is kept; this also caps
        // the 1/sin(theta') amplification of rounding at 100.
        if (sp >= R(1e-2)) {
          const R b = st / sp;
          const R a = ct - b * cp;
          nv[0] = a * sx + b * nv[0];
          nv[1] = a * sy + b * nv[1];
          nv[2] = a * sz + b * nv[2];
        }
      }
    }
  }
}

template <int P, bool LARGE>
__global__ __launch_bounds__(kBlock) void k_normal(StepArgs<P> A) {
  using R = typename Prec<P>::R;
  using D = D3Q19;
  using Off = typename Prec<P>::Off;
  const uint32_t t = uint32_t(run_block<LARGE>()) * kBlock + threadIdx.x;
  if (t >= uint32_t(A.nfluid)) return;
  const ListNode ln = ldx<Off>(A.fluid, t);
  const int n = ln.node;
  const uint32_t inf = ln.info;
  const Nbr nb = make_nbr(n, inf, A.geo);
  // The wetting data of a wetting node is loaded with the neighbours' colours, not after the
  // gradient: one memory round trip for the node instead of two.
  typename V4<R>::T wv;
  wv.x = wv.y = wv.z = wv.w = R(0);
  if (inf & kWet) wv = ld4<Off>(A.wet, t);
  R src[18];  // rho^N at x - c_i (solid neighbours hold their extrapolated colour)
  row_shared<false>(inf, ldx<Off>(A.rhoN, uint32_t(n)),
                    [&](int i) { return uint32_t(nb.at(-D::cx[i], -D::cy[i], -D::cz[i])); },
                    [&](uint32_t k) { return ldx<Off>(A.rhoN, k); }, [](int) { return true; }, src);
  R d[9];
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const int p = D::half[j];
    d[j] = rn_diff(src[D::opp[p]], src[p]);  // x + c_p is the source of opp(p)
  }
  R nv[3], len, raw[3];
  bool raw_set;
  for (int a = 0; a < 3; ++a) any_value(raw[a], a);  // read where raw_set
  normal_from_pairs<R>(d, inf, wv, A.eps, nv, len, raw, raw_set);
  if (raw_set && A.nraw) st4<Off>(A.nraw, t, raw[0], raw[1], raw[2], R(0));
  Vec3<R>& nst = ref3<Off>(A.nst, t);
  if (LARGE) {
    put<true>(nst.x, nv[0]);
    put<true>(nst.y, nv[1]);
    put<true>(nst.z, nv[2]);
    put<true>(refx<Off>(A.glen, t), len);
  } else {
    nst = {nv[0], nv[1], nv[2]};
    refx<Off>(A.glen, t) = len;
  }
}

// T^{-1} k* of Appendix A (eq. back_transformation_vector), regrouped with common
// subexpressions: for a move along +-x, q_x = u_x^2 +- u_x, and similarly for y, z.
template <class R>
__device__ inline void cm_back(R ux, R uy, R uz, R k5, R k6, R k7, R k8, R k9, R d[19]) {
  const R x2 = ux * ux, y2 = uy * uy, z2 = uz * uz;
  const R pxp = x2 + ux, pxm = x2 - ux, pyp = y2 + uy, pym = y2 - uy, pzp = z2 + uz, pzm = z2 - uz;
  const R ax = k5 * R(1.0 / 3.0) + k6 * R(1.0 / 6.0);
  const R ay = (k6 - k5) * R(1.0 / 6.0);
  const R az = -(k5 * R(1.0 / 6.0) + k6 * R(1.0 / 3.0));
  const R tx = uy * k7 + uz * k8, ty = ux * k7 + uz * k9, tz = ux * k8 + uy * k9;
  const R ux2 = ux + ux, uy2 = uy + uy, uz2 = uz + uz;
  d[0] = (pxp - y2 - z2 + R(1)) * ax - (ux2 + R(1)) * tx;
  d[1] = (pxm - y2 - z2 + R(1)) * ax - (ux2 - R(1)) * tx;
  d[2] = (pyp - x2 - z2 + R(1)) * ay - (uy2 + R(1)) * ty;
  d[3] = (pym - x2 - z2 + R(1)) * ay - (uy2 - R(1)) * ty;
  d[4] = (pzp - x2 - y2 + R(1)) * az - (uz2 + R(1)) * tz;
  d[5] = (pzm - x2 - y2 + R(1)) * az - (uz2 - R(1)) * tz;
  const R c12 = R(1.0 / 12.0), c4 = R(0.25);
  // xy plane: (-q_x + 2 q_y) k5 + (q_x + q_y) k6 + 3 (2u_x + s_x)(2u_y + s_y) k7, all / 12
  d[6] = ((pyp + pyp - pxp) * k5 + (pxp + pyp) * k6) * c12 + (ux2 + R(1)) * (uy2 + R(1)) * k7 * c4;
  d[7] = ((pym + pym - pxp) * k5 + (pxp + pym) * k6) * c12 + (ux2 + R(1)) * (uy2 - R(1)) * k7 * c4;
  d[10] = ((pyp + pyp - pxm) * k5 + (pxm + pyp) * k6) * c12 + (ux2 - R(1)) * (uy2 + R(1)) * k7 * c4;
  d[11] = ((pym + pym - pxm) * k5 + (pxm + pym) * k6) * c12 + (ux2 - R(1)) * (uy2 - R(1)) * k7 * c4;
  // xz plane: (-q_x + 2 q_z) k5 + (-2 q_x + q_z) k6 + 3 (2u_x + s_x)(2u_z + s_z) k8
  d[8] = ((pzp + pzp - pxp) * k5 + (pzp - pxp - pxp) * k6) * c12 + (ux2 + R(1)) * (uz2 + R(1)) * k8 * c4;
  d[9] = ((pzm + pzm - pxp) * k5 + (pzm - pxp - pxp) * k6) * c12 + (ux2 + R(1)) * (uz2 - R(1)) * k8 * c4;
  d[12] = ((pzp + pzp - pxm) * k5 + (pzp - pxm - pxm) * k6) * c12 + (ux2 - R(1)) * (uz2 + R(1)) * k8 * c4;
  d[13] = ((pzm + pzm - pxm) * k5 + (pzm - pxm - pxm) * k6) * c12 + (ux2 - R(1)) * (uz2 - R(1)) * k8 * c4;
  // yz plane: (-q_y - q_z) k5 + (-2 q_y + q_z) k6 + 3 (2u_y + s_y)(2u_z + s_z) k9
  d[14] = (-(pyp + pzp) * k5 + (pzp - pyp - pyp) * k6) * c12 + (uy2 + R(1)) * (uz2 + R(1)) * k9 * c4;
  d[15] = (-(pyp + pzm) * k5 + (pzm - pyp - pyp) * k6) * c12 + (uy2 + R(1)) * (uz2 - R(1)) * k9 * c4;
  d[16] = (-(pym + pzp) * k5 + (pzp - pym - pym) * k6) * c12 + (uy2 - R(1)) * (uz2 + R(1)) * k9 * c4;
  d[17] = (-(pym + pzm) * k5 + (pzm - pym - pym) * k6) * c12 + (uy2 - R(1)) * (uz2 - R(1)) * k9 * c4;
  d[18] = ((y2 + z2 - x2 - x2) * k5 + (z2 + z2 - x2 - y2) * k6) * R(1.0 / 3.0) +
          R(4) * (ux * uy * k7 + ux * uz * k8 + uy * uz * k9);
}

template <class R>
__device__ inline bool finite(R v) {
  return isfinite(v);
}

// Deterministic FP64 reduction over the workgroup of four sums and of the lanes with s[4] != 0: the
// wave's sums, then the workgroup's waves in fixed order; one partial per workgroup (plain stores, no
// fences or atomics). The sums are finished by reduce_partials, after the grid, in workgroup order.
template <int THREADS>
__device__ inline void block_reduce5(const double s[5], double* partials, int skip = 0) {
  __shared__ double red[kBlock / 64][5];
  const double v = wave_sums(s[0], s[1], s[2], s[3]);
  const int flagged = __popcll(__ballot(s[4] != 0));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane % 16 == 0) red[wave][lane / 16] = v;
  if (lane == 0) red[wave][4] = double(flagged);
  __syncthreads();
  if (threadIdx.x < 5) {
    double sum = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) sum += red[w][threadIdx.x];
    partials[size_t(threadIdx.x) * (gridDim.x - skip) + logical_block(skip)] = sum;
  }
}

// H |G| at fluid node x: the curvature H = -(tr J - n.J.n) (eq. interface_curvature) with
// J_ab = 3 sum_i w_i c_ib n*_a(x + c_i), times the gradient magnitude |G| of x; zero where
// |G| <= eps (no normal). nsv: (n*, |G|) of x; nbr(i): n* at x + c_i, or of x itself where x + c_i is
// solid (the value the curvature takes for a solid neighbour). Every pass that forms the
// curvature calls this.
template <class R, class NbrN>
__device__ inline R curvature_hg(const typename V4<R>::T& nsv, R eps, NbrN nbr) {
  using D = D3Q19;
  R J[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
  for (int i = 0; i < 18; ++i) {
    const Vec3<R> nbi = nbr(i);
    const R a0 = nbi.x, a1 = nbi.y, a2 = nbi.z;
    const R w3 = R(3.0 * D::w(i));
    if (D::cx[i]) { J[0][0] += w3 * R(D::cx[i]) * a0; J[1][0] += w3 * R(D::cx[i]) * a1; J[2][0] += w3 * R(D::cx[i]) * a2; }
    if (D::cy[i]) { J[0][1] += w3 * R(D::cy[i]) * a0; J[1][1] += w3 * R(D::cy[i]) * a1; J[2][1] += w3 * R(D::cy[i]) * a2; }
    if (D::cz[i]) { J[0][2] += w3 * R(D::cz[i]) * a0; J[1][2] += w3 * R(D::cz[i]) * a1; J[2][2] += w3 * R(D::cz[i]) * a2; }
  }
  const R glen = nsv.w;
  R H = 0;
  if (glen > eps) {
    const R nn[3] = {nsv.x, nsv.y, nsv.z};
    R nJn = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) nJn += nn[a] * nn[b] * J[a][b];
    H = -((J[0][0] + J[1][1] + J[2][2]) - nJn);
  }
  return H * glen;
}

// One value to each of K planes.
template <bool STREAM, class Off, int K, class S>
__device__ inline void put_planes(S* planes, size_t ps, uint32_t t, const S (&v)[K]) {
#pragma unroll
  for (int i = 0; i < K; ++i) put<STREAM>(refx<Off>(planes + size_t(i) * ps, t), v[i]);
}

// The collision and the rest of the step at one fluid node x (fluid id t, node n, info word inf):
// moments, forcing, central-moment collision, recolouring, reaction, species, store, and the
// node's contribution to the FP64 sums (added to red5). f, g: the pulled populations; rn: rho^N(x)
// (rn_value form); cur: (n*, H |G|) of x (n* = 0 where x has no normal). MOM writes the level-t
// fields instead.
template <int P, bool MOM, int STREAM>
__device__ inline void collide_node(const StepArgs<P>& A, uint32_t t, int n, uint32_t inf,
                                    const typename Prec<P>::R f[19], const typename Prec<P>::R g[7],
                                    typename Prec<P>::R rn, const typename V4<typename Prec<P>::R>::T& cur,
                                    double red5[5]) {
  using R = typename Prec<P>::R;
  using Off = typename Prec<P>::Off;
  using D = D3Q19;
  const size_t N = A.N;
  // Moments (same summation order as k_colour, so rho^m agrees bit for bit).
  R rm = 0;
#pragma unroll
  for (int i = 0; i < 19; ++i) rm += f[i];
  R mx = 0, my = 0, mz = 0, pxx = 0, pyy = 0, pzz = 0, pxy = 0, pxz = 0, pyz = 0;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    if (D::cx[i]) { mx += R(D::cx[i]) * f[i]; pxx += f[i]; }
    if (D::cy[i]) { my += R(D::cy[i]) * f[i]; pyy += f[i]; }
    if (D::cz[i]) { mz += R(D::cz[i]) * f[i]; pzz += f[i]; }
    if (D::cx[i] && D::cy[i]) pxy += R(D::cx[i] * D::cy[i]) * f[i];
    if (D::cx[i] && D::cz[i]) pxz += R(D::cx[i] * D::cz[i]) * f[i];
    if (D::cy[i] && D::cz[i]) pyz += R(D::cy[i] * D::cz[i]) * f[i];
  }
  const R irm = R(1) / rm;
  const R ux = mx * irm, uy = my * irm, uz = mz * irm;
  R rr, rp;
  rn_densities(rn, rm, rr, rp);

  // Realigned unit normal (zero where the node has no normal: a unit vector otherwise) and the
  // exact-difference forcing du^k = F^k / rho^k = (1/2) sigma H |G| n* / rho^m + a^k.
  const R n0 = cur.x, n1 = cur.y, n2 = cur.z;
  const bool has_n = n0 != R(0) || n1 != R(0) || n2 != R(0);
  const R fc = R(0.5) * A.sigma * cur.w * irm;
  const R dur[3] = {fc * n0 + A.acc[0][0], fc * n1 + A.acc[0][1], fc * n2 + A.acc[0][2]};
  const R dup[3] = {fc * n0 + A.acc[1][0], fc * n1 + A.acc[1][1], fc * n2 + A.acc[1][2]};
  const R upx = ux + R(0.5) * (rr * dur[0] + rp * dup[0]) * irm;
  const R upy = uy + R(0.5) * (rr * dur[1] + rp * dup[1]) * irm;
  const R upz = uz + R(0.5) * (rr * dur[2] + rp * dup[2]) * irm;

  R C = R(1);
  if (A.species) {
    C = 0;
#pragma unroll
    for (int i = 0; i < 7; ++i) C += g[i];
    if (inf & kInlet) C = A.c_in;
  }

  if (MOM) {
    if (A.m_rr) A.m_rr[n] = rr;
    if (A.m_rp) A.m_rp[n] = rp;
    if (A.m_rn) A.m_rn[n] = rn_value(rn);
    if (A.m_u) { A.m_u[n] = upx; A.m_u[N + n] = upy; A.m_u[2 * N + n] = upz; }
    if (A.m_c) A.m_c[n] = C;
  } else {
    // Central shear moments k5..k9 about the bare velocity, relaxed by (1 - 1/tau).
    const R cxx = pxx - rm * ux * ux, cyy = pyy - rm * uy * uy, czz = pzz - rm * uz * uz;
    const R k5 = A.relax * (cxx - cyy), k6 = A.relax * (cyy - czz);
    const R k7 = A.relax * (pxy - rm * ux * uy), k8 = A.relax * (pxz - rm * ux * uz), k9 = A.relax * (pyz - rm * uy * uz);
    R d[19];
    cm_back(ux, uy, uz, k5, k6, k7, k8, k9, d);
    // f^{m,*} = f^eq(rho^r, u + du^r) + f^eq(rho^p, u + du^p) + T^{-1} k*: the sum of both
    // colours' equilibria needs only M = sum_k rho^k U^k and Pi = sum_k rho^k U^k U^k.
    const R Ur[3] = {ux + dur[0], uy + dur[1], uz + dur[2]};
    const R Up[3] = {ux + dup[0], uy + dup[1], uz + dup[2]};
    const R M0 = rr * Ur[0] + rp * Up[0], M1 = rr * Ur[1] + rp * Up[1], M2 = rr * Ur[2] + rp * Up[2];
    const R Pxx = rr * Ur[0] * Ur[0] + rp * Up[0] * Up[0];
    const R Pyy = rr * Ur[1] * Ur[1] + rp * Up[1] * Up[1];
    const R Pzz = rr * Ur[2] * Ur[2] + rp * Up[2] * Up[2];
    const R Pxy = rr * Ur[0] * Ur[1] + rp * Up[0] * Up[1];
    const R Pxz = rr * Ur[0] * Ur[2] + rp * Up[0] * Up[2];
    const R Pyz = rr * Ur[1] * Ur[2] + rp * Up[1] * Up[2];
    const R base = rm - R(1.5) * (Pxx + Pyy + Pzz);
    R fs[19];
    R fsum = 0;
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      const int cx = D::cx[i], cy = D::cy[i], cz = D::cz[i];
      R cM = 0, cPc = 0;
      if (cx) { cM += R(cx) * M0; cPc += Pxx; }
      if (cy) { cM += R(cy) * M1; cPc += Pyy; }
      if (cz) { cM += R(cz) * M2; cPc += Pzz; }
      if (cx && cy) cPc += R(2 * cx * cy) * Pxy;
      if (cx && cz) cPc += R(2 * cx * cz) * Pxz;
      if (cy && cz) cPc += R(2 * cy * cz) * Pyz;
      fs[i] = R(D::w(i)) * (base + R(3) * cM + R(4.5) * cPc) + d[i];
      fsum += fs[i];
    }
    // Wall reaction with level-t densities, capped at full conversion.
    const int rnn = int((inf & kRnnMask) >> kRnnShift);
    R delta = 0;
    if (rnn > 0 && rr > R(0)) {
      if (A.species) {
        if (C > R(0)) {
          const R rate = A.xi * R(rnn) * rr * C;
          const R cap = fmin(rr, C);
          delta = fmin(rate, cap);
        }
      } else {
        delta = fmin(A.xi * R(rnn), R(1)) * rr;
      }
    }
    const R keep = (delta != R(0)) ? R(1) - delta / rr : R(1);
    // Compact recoloured state: a = (rho^r - delta)/rho^m, b = (rho^p + delta)/rho^m,
    // v = keep beta rho^r rho^p/rho^m n* with keep = 1 - delta/rho^r.
    const R aout = pack_frac((rr - delta) * irm, (rp + delta) * irm);
    const R vc = keep * A.beta * rr * rp * irm;
    const R v0 = has_n ? vc * n0 : R(0), v1 = has_n ? vc * n1 : R(0), v2 = has_n ? vc * n2 : R(0);
    typename Prec<P>::S fo[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) fo[i] = Prec<P>::st(fs[i], R(D::w(i)), A.scale);
    put_planes<STREAM == 2, Off>(A.fout, A.ps, t, fo);
    if (STREAM == 2 && A.stream_vectors) {
      keep_apart();
      st4_stream<Off>(A.aout, t, aout, v0, v1, v2);
      keep_apart();
    } else {
      st4<Off>(A.aout, t, aout, v0, v1, v2);
    }
    bool ok = finite(fsum) && finite(aout) && finite(v0 + v1 + v2) && finite(rr) && finite(rp);
    if (A.species) {
      // BGK towards g^eq = w C (1 + 4 c.u_phys); at the inlet the populations are replaced by
      // the equilibrium at C_in; then the reaction sink.
      const bool inlet = inf & kInlet;
      const R sink = (delta != R(0)) ? R(1) - delta / C : R(1);
      const R cu[7] = {upx, -upx, upy, -upy, upz, -upz, R(0)};
      R go[7];
      R gs = 0;
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        const R geq = R(D3Q7::w(i)) * C * (R(1) + R(4) * cu[i]);
        const R gi = inlet ? geq : g[i];
        go[i] = (gi + (geq - gi) * A.inv_tau_c) * sink;
        gs += go[i];
      }
      if (Prec<P>::deviations) refx<Off>(A.cout, t) = gs;  // the deviation reference of the stored populations
      typename Prec<P>::S gq[7];
#pragma unroll
      for (int i = 0; i < 7; ++i) gq[i] = Prec<P>::st(go[i], Prec<P>::deviations ? R(D3Q7::w(i)) * gs : R(D3Q7::w(i)), A.gscale);
      put_planes<STREAM != 0, Off>(A.gout, A.ps, t, gq);
      ok = ok && finite(gs);
    }
    red5[0] += double(rr);
    red5[1] += double(rp);
    red5[2] += double(delta);
    red5[3] += double(C);
    red5[4] += ok ? 0.0 : 1.0;
  }
}

// ---------------------------------------------------------------------------------------------
// collide: the rest of the step at every fluid node. MOM = true writes the level-t fields
// instead (lbm_moments) and leaves the state untouched. Four waves per SIMD in FP32, FP16 and BF16
// (at most 128 VGPRs, no spills; a five-wave bound made the 2-byte storages spill and run 11%
// slower at 512^3); FP64 runs fewer.
//
// IFACE = true: rho^N and the realigned normals come from the colour and normal passes. A wave none
// of whose nodes has |G| > eps skips its neighbours' normals: H is zero there whatever they are (the
// own (n*, |G|) is loaded with the list entry, so the test costs no round trip; the sweep's 128^3
// set-up, with interfaces round eight nucleation sites, 43 -> 40 us, waves without such nodes the same). IFACE = false, chosen
// when sigma = beta = 0: neither the force nor the recolouring uses a normal, rho^N is needed at the
// node alone, and this one kernel is the whole step, forming rho^N from its own pull.
// STREAM: nontemporal stores of the species (1) or of all populations (2).
// ---------------------------------------------------------------------------------------------
template <int P, bool MOM, bool IFACE, int THREADS, int STREAM>
__global__ __launch_bounds__(THREADS) void k_collide(StepArgs<P> A) {
  using R = typename Prec<P>::R;
  using D = D3Q19;
  using Off = typename Prec<P>::Off;
  if (!IFACE && finish_previous<THREADS>(A)) return;
  const int skip = !IFACE && A.red_out ? kXcd : 0;
  const uint32_t t = split_tile_id<THREADS, false>(A, skip);
  double red5[5] = {0, 0, 0, 0, 0};
  if (t < uint32_t(A.nfluid)) {
    const ListNode ln = ldx<Off>(A.fluid, t);
    typename V4<R>::T own;  // (n*, |G|) of the node, or its colour scalars (e, v)
    Vec3<R> own_n;
    if (IFACE) {
      own_n = ld3<Off>(A.nst, t);
      own.x = own_n.x; own.y = own_n.y; own.z = own_n.z;
      own.w = ldx<Off>(A.glen, t);
    } else {
      own = ld4<Off>(A.ain, t);
    }
    const int n = ln.node;
    const uint32_t inf = ln.info;
    const Nbr nb = make_nbr(n, inf, A.geo);
    // All loads of the node together (pull of f^m and g with halfway bounce-back, rho^N, the
    // neighbours' vectors), so that one memory round trip covers them.
    uint32_t sid[18];  // fluid ids of the pull sources (own id for bounce-back)
    pull_sources<Off>(A.ids, nb, t, inf, sid);
    typename Prec<P>::S s[19];
    ld_populations(A, t, inf, sid, s);
    R f[19], g[7];
    pull_species(A, t, inf, sid, g);
    R rn = 0;
    if (IFACE) rn = ldx<Off>(A.rhoN, uint32_t(n));
    const RowLanes lanes = row_lanes(inf);
    const auto idx = [&](int i) { return sid[i]; };
    const auto all = [](int) { return true; };
    typename V4<R>::T cur;
    cur.x = cur.y = cur.z = cur.w = 0;
    if (IFACE) {
      cur = own;
      cur.w = R(0) * own.w;
      if (__any(own.w > A.eps)) {
        // x + c_i is the pull source of direction opp(i), the node's own id where it is solid, which
        // is the value the curvature takes for a solid neighbour.
        const auto ld = [&](uint32_t k) { return ld3<Off>(A.nst, k); };
        Vec3<R> nbr[18], edge[5];
        row_gather<true>(lanes, inf, idx, ld, all, nbr, edge);
        row_resolve<true>(lanes, inf, own_n, idx, ld, all, nbr, edge);
        cur.w = curvature_hg<R>(own, A.eps, [&](int i) { return nbr[D::opp[i]]; });
      }
#pragma unroll
      for (int i = 0; i < 19; ++i) f[i] = Prec<P>::ld(s[i], R(D::w(i)), A.inv_scale);
    } else {
      const auto ld = [&](uint32_t k) { return ld4<Off>(A.ain, k); };
      typename V4<R>::T nbr[18], edge[5];
      row_gather<true>(lanes, inf, idx, ld, all, nbr, edge);
      __builtin_amdgcn_sched_barrier(0);
      use_whole(nbr, edge);
      row_resolve<false>(lanes, inf, own, idx, ld, all, nbr, edge);
#pragma unroll
      for (int i = 0; i < 19; ++i) f[i] = Prec<P>::ld(s[i], R(D::w(i)), A.inv_scale);
      R rm;
      rn = colour_of<R>(inf, own, nbr, [&](int i) { return f[i]; }, rm);
    }
    collide_node<P, MOM, STREAM>(A, t, n, inf, f, g, rn, cur, red5);
  }
  if (!MOM && A.partials) block_reduce5<THREADS>(red5, A.partials, skip);
}

// Zeros for the fields of lbm_moments (any may be null), whose fluid nodes the collide pass then writes: at the
// solid nodes, or with info = null at every node. Whole lines take no info words and stream; the solid
// nodes alone write less where they are few (clears_whole in lbm.hip).
template <class R>
__global__ __launch_bounds__(kBlock) void k_clear(const uint32_t* info, int N, R* rr, R* rp, R* rn, R* u, R* c) {
  const size_t n = size_t(blockIdx.x) * kBlock + threadIdx.x, count = size_t(N);
  if (n >= count || (info && (info[n] & kFluid))) return;
  if (rr) rr[n] = R(0);
  if (rp) rp[n] = R(0);
  if (rn) rn[n] = R(0);
  if (u) u[n] = u[count + n] = u[2 * count + n] = R(0);
  if (c) c[n] = R(0);
}

// ---------------------------------------------------------------------------------------------
// FP64 sums of a stored state S_t: m^r = sum a rho_s, m^p = sum b rho_s (eqs. reactant_mass,
// product_mass), sum C_s and the non-finite count, with rho_s = sum_i f^m_i and C_s = sum_i g_i
// the node's stored totals. Every stored population is pulled exactly once (by its neighbour,
// or by the node itself through bounce-back), and the recolouring terms of a node cancel in
// opposite pairs, so these are the colour masses and species total of level t. Slot 2
// (conversion) is zero. One partial per workgroup, summed by k_finish_reduce.
// ---------------------------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(kBlock) void k_state_sums(StepArgs<P> A) {
  using R = typename Prec<P>::R;
  using D = D3Q19;
  using Off = typename Prec<P>::Off;
  const uint32_t t = uint32_t(logical_block()) * kBlock + threadIdx.x;
  double red5[5] = {0, 0, 0, 0, 0};
  if (t < uint32_t(A.nfluid)) {
    R a, b;
    unpack_frac(ld4<Off>(A.ain, t).x, a, b);
    R s = 0;
#pragma unroll
    for (int i = 0; i < 19; ++i)
      s += Prec<P>::ld(ldx<Off>(A.fin + size_t(i) * A.ps, t), R(D::w(i)), A.inv_scale);
    R C = 0;
    if (A.species)
#pragma unroll
      for (int i = 0; i < 7; ++i) C += ld_species(A, i, t);
    red5[0] = double(a) * double(s);
    red5[1] = double(b) * double(s);
    red5[3] = double(C);
    red5[4] = (finite(s) && finite(a) && finite(C)) ? 0.0 : 1.0;
  }
  block_reduce5<kBlock>(red5, A.partials);
}

// ---------------------------------------------------------------------------------------------
// Expansion of the stored state to per-colour populations (lbm_populations).
// ---------------------------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(kBlock) void k_expand(StepArgs<P> A, typename Prec<P>::R* fr,
                                                   typename Prec<P>::R* fp, typename Prec<P>::R* go) {
  using R = typename Prec<P>::R;
  using D = D3Q19;
  const int n = logical_block() * kBlock + threadIdx.x;
  if (n >= A.N) return;
  const size_t N = A.N;
  using Off = typename Prec<P>::Off;
  const IdWord word = A.ids[n >> 5];
  const bool fluid = is_fluid(word, uint32_t(n));
  const uint32_t fi = fluid ? fluid_before(word, uint32_t(n)) : 0;
  // Every load of the node before the first store (a solid node loads nothing), and the id word, which holds the
  // fluid bit, instead of an info word beside it: FP32 128^3 131 -> 116 us, 256^3 1030 -> 855; FP16 128^3 126 -> 106.
  typename V4<R>::T av;
  av.x = av.y = av.z = av.w = R(0);
  R fm[19], g[7];
#pragma unroll
  for (int i = 0; i < 19; ++i) fm[i] = R(0);
#pragma unroll
  for (int i = 0; i < 7; ++i) g[i] = R(0);
  if (fluid) {
    av = ld4<Off>(A.ain, fi);
#pragma unroll
    for (int i = 0; i < 19; ++i) fm[i] = Prec<P>::ld(ldx<Off>(A.fin + size_t(i) * A.ps, fi), R(D::w(i)), A.inv_scale);
    if (go && A.species)
#pragma unroll
      for (int i = 0; i < 7; ++i) g[i] = ld_species(A, i, fi);
  }
  const R v0 = av.y, v1 = av.z, v2 = av.w;
  R a, b;
  unpack_frac(av.x, a, b);
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    const R kv = R(D::w_over_len(i)) * (R(D::cx[i]) * v0 + R(D::cy[i]) * v1 + R(D::cz[i]) * v2);
    fr[size_t(i) * N + n] = fluid ? a * fm[i] + kv : R(0);
    fp[size_t(i) * N + n] = fluid ? b * fm[i] - kv : R(0);
  }
  if (go) {
#pragma unroll
    for (int i = 0; i < 7; ++i) go[size_t(i) * N + n] = g[i];
  }
}

}  // namespace lbm
