// Connected components (gfx950) and the pointer-forest compression entry.
//
// arXiv 2409.03771, Alg. 3 and methods "Connected Components": masked
// vertices point to a masked neighbour chosen by id, path compression turns
// the pointers into per-component labels, and a stitching step merges the
// partial trees that touch before a last compression.  Every pointer here
// goes to a smaller (or equal) id, so a component ends up named by its
// smallest id.  The paper's single racy stitch does not join every pair of
// touching trees in general; here trees are joined with a lock-free union
// (compare-and-swap of the larger root onto the smaller one, retried until
// it sticks), whose result is the min-id labelling whatever the schedule.
//
// Grid masks use the same two levels as the segmentation, mirroring the
// paper's rank-local pass plus exchange:
//   cc_tile    one workgroup per tile, one thread per row: union-find in LDS
//              over the rows' runs of masked vertices; writes the rows as bits
//              and each run's tile-local root (16-bit), and makes every
//              tile-local root its own parent in the global label array;
//   cc_cross   unions across the tile faces (each cross-tile edge once, from
//              the tile holding its lower endpoint) on the global array,
//              touching tile-local roots only (the paper's ghost exchange);
//   cc_final   label = root of the vertex's run's tile-local root.
// CSR graphs have no locality to exploit: hooks to a smaller masked neighbour,
// single attempts to join trees across sampled edges, a bitmap of the largest
// tree, unions along the listed edges that it does not settle, then a final
// walk per vertex.
#include <algorithm>
#include <climits>
#include <mutex>

#include "msc_internal.hpp"

namespace msc {
namespace {

__device__ __forceinline__ int64_t gid() {
  return (int64_t)blockIdx.x * kBlock + threadIdx.x;
}

__device__ __forceinline__ void flag_any(bool pred, unsigned long long *ctr) {
  if (__ballot(pred) && (threadIdx.x & 63) == 0) atomicOr(ctr, 1ull);
}

// ---------------------------------------------------------------------------
// Lock-free union-find on a parent array whose pointers only decrease.
// ---------------------------------------------------------------------------

template <class T>
__device__ __forceinline__ T uf_find(T *par, T x) {
  for (;;) {
    T p = __atomic_load_n(&par[x], __ATOMIC_RELAXED);
    if (p == x) return x;
    T g = __atomic_load_n(&par[p], __ATOMIC_RELAXED);
    if (g == p) return p;
    // Path halving: g is an ancestor of x, so this only shortens the path.
    __atomic_store_n(&par[x], g, __ATOMIC_RELAXED);
    x = g;
  }
}

// Root of x without writing: used once no union is running, by the passes
// in which every entry is also an output that only its owner may write.
// The loads are cached (workgroup scope): a value older than another
// workgroup's write is still an ancestor on the path to the same root.
template <class T>
__device__ __forceinline__ T uf_root(const T *par, T x) {
  for (;;) {
    T p = __hip_atomic_load(&par[x], __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_WORKGROUP);
    if (p == x) return x;
    x = p;
  }
}

// Join the trees of a and b: the larger root is hung under the smaller one.
template <class T>
__device__ __forceinline__ bool uf_unite(T *par, T a, T b) {
  bool changed = false;
  for (;;) {
    a = uf_find(par, a);
    b = uf_find(par, b);
    if (a == b) return changed;
    if (a > b) {
      T t = a;
      a = b;
      b = t;
    }
    T expect = b;
    if (__atomic_compare_exchange_n(&par[b], &expect, a, false,
                                    __ATOMIC_RELAXED, __ATOMIC_RELAXED))
      return true;
    changed = true;  // b moved meanwhile; retry from the new trees
  }
}

// The same on a forest in device memory, where every step of a walk is a
// round trip: the two walks of a union advance side by side (each step's
// loads for both are issued before either is used; a walk that has reached
// its root reloads it harmlessly), and the accesses are at device scope,
// which is all that one device's workgroups need.
template <class T>
__device__ __forceinline__ T ld_dev(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T>
__device__ __forceinline__ void uf_find2_dev(T *par, T &a, T &b) {
  bool ra = false, rb = false;
  while (!(ra && rb)) {
    const T pa = ld_dev(&par[a]), pb = ld_dev(&par[b]);
    const T ga = ld_dev(&par[pa]), gb = ld_dev(&par[pb]);
    if (!ra) {
      if (pa == a) {
        ra = true;
      } else if (ga == pa) {
        a = pa;
        ra = true;
      } else {
        // Path halving: ga is an ancestor of a, so this only shortens it.
        __hip_atomic_store(&par[a], ga, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        a = ga;
      }
    }
    if (!rb) {
      if (pb == b) {
        rb = true;
      } else if (gb == pb) {
        b = pb;
        rb = true;
      } else {
        __hip_atomic_store(&par[b], gb, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        b = gb;
      }
    }
  }
}

template <class T>
__device__ __forceinline__ void uf_unite_dev(T *par, T a, T b) {
  for (;;) {
    uf_find2_dev(par, a, b);
    if (a == b) return;
    if (a > b) {
      const T t = a;
      a = b;
      b = t;
    }
    T expect = b;
    if (__hip_atomic_compare_exchange_strong(
            &par[b], &expect, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
            __HIP_MEMORY_SCOPE_AGENT))
      return;  // otherwise b moved meanwhile; retry from the new trees
  }
}

// ---------------------------------------------------------------------------
// Grid masks
// ---------------------------------------------------------------------------

constexpr int CTX = 32, CTY = 16, CTZ = 16;      // tile
constexpr int kCThreads = CTX * CTY;             // the label pass: one per column
constexpr int kCOwned = CTX * CTY * CTZ;
static_assert(kCOwned < 65535, "tile-local roots are 16-bit");

struct CGeo {
  int64_t X, Y, Z, XY, N;
  int64_t ntx, nty, ntz;
};

__device__ __forceinline__ uint32_t cc_tile_of_block(uint32_t b, uint32_t nb) {
  const uint32_t per = nb / 8, rem = nb % 8, xcd = b % 8, idx = b / 8;
  return xcd < rem ? xcd * (per + 1) + idx
                   : rem * (per + 1) + (xcd - rem) * per + idx;
}

struct CTile {
  int64_t x0, y0, z0;
};

__device__ __forceinline__ CTile ctile_at(const CGeo &g, int64_t t) {
  int64_t tx = t % g.ntx, r = t / g.ntx;
  int64_t ty = r % g.nty, tz = r / g.nty;
  return CTile{tx * CTX, ty * CTY, tz * CTZ};
}

// What a tile's own pass leaves for the other two, in the tile's slot of the
// workspace (kCOwned 16-bit words, of which 6.5 KB stay unused): its
// rows as 32-bit masks, the number of each row's first run, and for every run
// (consecutive masked x of a row, numbered in index order) the local index of
// its component's first vertex.  A row is CTX vertices; row r = ly + CTY*lz.
constexpr int kCRows = CTY * CTZ;
constexpr int kCRuns = kCRows * (CTX / 2);  // at most 16 runs in 32 bits
static_assert(CTX == 32, "a row is one word");

struct CTileOut {
  uint32_t word[kCRows];
  uint16_t base[kCRows];
  uint16_t root[kCRuns];
};
static_assert(sizeof(CTileOut) <= kCOwned * sizeof(uint16_t), "fits the slot");

__device__ __forceinline__ CTileOut *ctile_out(uint16_t *loc, int64_t t) {
  return reinterpret_cast<CTileOut *>(loc + t * kCOwned);
}

// First and last bits of a word's runs, and the number of the run that holds
// bit x among them.
__device__ __forceinline__ uint32_t run_starts(uint32_t w) {
  return w & ~(w << 1);
}
__device__ __forceinline__ uint32_t run_ends(uint32_t w) {
  return w & ~(w >> 1);
}
__device__ __forceinline__ uint32_t run_of(uint32_t starts, int x) {
  return (uint32_t)__popc(starts & (0xffffffffu >> (31 - x))) - 1u;
}

// Global id of the tile-local index l (lx + CTX*(ly + CTY*lz)).
__device__ __forceinline__ int64_t ctile_global(const CGeo &g, const CTile &t,
                                                int l) {
  const int lz = l / (CTX * CTY), r = l - lz * (CTX * CTY);
  const int ly = r / CTX, lx = r - ly * CTX;
  return (t.x0 + lx) + g.X * (t.y0 + ly) + g.XY * (t.z0 + lz);
}

// One mask of a launch: its buffers, shape and first tile.  A launch covers
// the tiles of up to B masks (B = 1 for a single mask), passed by value.
struct CGrid {
  const uint8_t *mask;
  int64_t *L;      // labels, also the union-find parent array
  uint16_t *loc;   // the tiles' slots (workspace): ctile_out
  int64_t off;     // added to every label (a slab inside a larger grid)
  int64_t X, Y, Z;
  uint32_t tile0;  // first tile of this mask in the launch
};

template <int B>
struct CBatch {
  int n;
  CGrid g[B];
};

// The mask and geometry of launch tile `tt`, and the tile's index within it.
template <int B>
__device__ __forceinline__ const CGrid &cgrid_of(const CBatch<B> &b,
                                                 uint32_t tt, CGeo *g,
                                                 int64_t *t) {
  int lo = 0;
  if (B > 1) {
    int hi = b.n - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (b.g[mid].tile0 <= tt) lo = mid;
      else hi = mid - 1;
    }
  }
  const CGrid &d = b.g[lo];
  const int64_t X = d.X, Y = d.Y, Z = d.Z;
  *g = CGeo{X, Y, Z, X * Y, X * Y * Z, (X + CTX - 1) / CTX,
            (Y + CTY - 1) / CTY, (Z + CTZ - 1) / CTZ};
  *t = (int64_t)(tt - d.tile0);
  return d;
}

// 32 mask bytes from p as bits (any alignment; they must exist).
__device__ __forceinline__ uint32_t mask_bits32(const uint8_t *p) {
  struct __attribute__((packed)) Bytes {
    uint32_t w[8];
  };
  const Bytes b = *reinterpret_cast<const Bytes *>(p);
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    // The top bit of every byte that is not zero, then those four together.
    const uint32_t t = (((b.w[k] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | b.w[k]) &
                       0x80808080u;
    m |= (((t >> 7) * 0x01020408u) >> 24) << (4 * k);
  }
  return m;
}

// One thread per row.  A row's runs of masked x are the nodes: joining them
// settles every x edge, and the edges between two rows are joined once per
// pair of runs that touch, found with a few operations on the rows' words,
// whatever the number of vertices.  What bounds the pass is the latency of its
// steps (load, scan, unions in LDS, stores), so a tile holds four waves and a
// CU six tiles.  At 1024^3 with 30 % in the mask it takes 0.40 ms (0.43 where
// every pair of runs is joined and none starts under another); with a thread
// per column, which loads its bytes one by one and unites vertex by vertex, it
// took 2.0.  Rows of many runs are the slow ones: every other vertex masked in
// all three directions takes 0.13 ms at 256^3, columns of every other x joined by
// full rows 0.10 (0.04 with a thread per column).
constexpr int kCTileThreads = kCRows;

template <int B>
__global__ void __launch_bounds__(kCTileThreads) k_cc_tile(CBatch<B> b) {
  __shared__ int32_t par[kCRuns];
  __shared__ uint16_t head[kCRuns];        // local index of a run's first vertex
  __shared__ uint32_t word[kCRows], base[kCRows];
  __shared__ uint32_t wsum[kCTileThreads / 64];
  const int r = threadIdx.x, lane = r & 63, wave = r >> 6;
  CGeo g;
  int64_t ti;
  const CGrid &d = cgrid_of(b, cc_tile_of_block(blockIdx.x, gridDim.x), &g,
                            &ti);
  const CTile t = ctile_at(g, ti);
  const int ly = r % CTY, lz = r / CTY;
  const int64_t gy = t.y0 + ly, gz = t.z0 + lz;
  uint32_t m = 0;
  if (gy < g.Y && gz < g.Z) {
    const int64_t at = t.x0 + g.X * gy + g.XY * gz;
    const int nx = (int)(g.X - t.x0 < CTX ? g.X - t.x0 : CTX);
    if (at + CTX <= g.N) {
      m = mask_bits32(d.mask + at) & (0xffffffffu >> (CTX - nx));
    } else {  // the mask's last rows: no byte past its end
      for (int x = 0; x < nx; ++x) m |= (uint32_t)(d.mask[at + x] != 0) << x;
    }
  }
  // Run numbers: an exclusive scan of the rows' counts.
  const uint32_t st = run_starts(m), cnt = (uint32_t)__popc(st);
  uint32_t inc = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  word[r] = m;
  __syncthreads();
  uint32_t first = inc - cnt, runs = 0;
#pragma unroll
  for (int w = 0; w < kCTileThreads / 64; ++w) {
    first += w < wave ? wsum[w] : 0u;
    runs += wsum[w];
  }
  base[r] = first;
  {
    uint32_t i = first;
    for (uint32_t s = st; s; s &= s - 1, ++i)
      head[i] = (uint16_t)(r * CTX + __ffs((int)s) - 1);
  }
  __syncthreads();
  // Edges to the rows before (y-1), (z-1) and (y-1, z-1): x touches x and x-1
  // there.  A run A = [a, b] and a run B = [c, e] of the other row touch when
  // c <= b and e >= a - 1: they overlap from max(a, c) on, where one of them
  // starts, or B ends just before a; there is one such position for every pair
  // of runs that touch.  An edge into the diagonal row is implied where x is
  // masked in one of the other two rows.
  const uint32_t ny = m && ly > 0 ? word[r - 1] : 0u;
  const uint32_t nz = m && lz > 0 ? word[r - CTY] : 0u;
  const uint32_t nd = m && ly > 0 && lz > 0 ? word[r - CTY - 1] : 0u;
  auto touch = [&](uint32_t nw) {
    return (m & nw & (st | run_starts(nw))) | (st & ~nw & (nw << 1));
  };
  // Number of the run of row `row` (word nw) that is touched at position x.
  auto touched = [&](uint32_t nw, int row, int x) {
    return base[row] + run_of(run_starts(nw), (nw >> x) & 1u ? x : x - 1);
  };
  // The positions of c that are the first in their run of this row.
  auto firsts = [&](uint32_t c) {
    uint32_t f = c, p = m;
#pragma unroll
    for (int k = 1; k < 32; k <<= 1) {
      f |= p & (f << k);
      p &= p << k;
    }
    return c & ~(m & (f << 1));
  };
  // A run starts under the first one that it touches, which has a smaller
  // number: half of the joins at the price of a store.
  uint32_t cy = touch(ny), cz = touch(nz), hooked = 0;
  {
    const uint32_t f = firsts(cy);
    cy &= ~f;
    for (uint32_t c = f; c; c &= c - 1) {
      const int x = __ffs((int)c) - 1;
      const uint32_t k = run_of(st, x);
      hooked |= 1u << k;
      par[first + k] = (int32_t)touched(ny, r - 1, x);
    }
  }
  for (uint32_t c = firsts(cz); c; c &= c - 1) {
    const int x = __ffs((int)c) - 1;
    const uint32_t k = run_of(st, x);
    if ((hooked >> k) & 1u) continue;
    hooked |= 1u << k;
    cz &= ~(1u << x);
    par[first + k] = (int32_t)touched(nz, r - CTY, x);
  }
  for (uint32_t k = 0; k < cnt; ++k)
    if (!((hooked >> k) & 1u)) par[first + k] = (int32_t)(first + k);
  __syncthreads();
  auto join = [&](uint32_t c, uint32_t nw, int row) {
    for (; c; c &= c - 1) {
      const int x = __ffs((int)c) - 1;
      uf_unite<int32_t>(par, (int32_t)(first + run_of(st, x)),
                        (int32_t)touched(nw, row, x));
    }
  };
  join(cy, ny, r - 1);
  join(cz, nz, r - CTY);
  join(touch(nd) & ~(ny | nz), nd, r - CTY - 1);
  __syncthreads();
  CTileOut *out = ctile_out(d.loc, ti);
  out->word[r] = m;
  out->base[r] = (uint16_t)first;
  for (uint32_t i = r; i < runs; i += kCTileThreads) {
    const int32_t root = uf_find<int32_t>(par, (int32_t)i);
    out->root[i] = head[root];
    if (root == (int32_t)i) {  // tile-local roots start as global roots
      const int64_t v = ctile_global(g, t, head[i]);
      d.L[v] = v;
    }
  }
}

// Unions across tile faces.  An edge between two tiles is handled by the tile
// that owns its lower endpoint, which sees it as one of the 7 higher-id
// neighbours leaving the tile through an upper face.  Both ends' runs are
// replaced by their tile-local roots, and each distinct (local root, neighbour
// tile, its local root) triple is united once, after the block has collected
// them: a face of a smooth mask carries thousands of edges but only a few such
// triples.  One thread per row, on the words of the tile's rows, of the rows
// just beyond it, and of the tiles one up in x: 2.3 KB in a few whole lines,
// where a 16-bit entry per vertex of the faces touched every line of the
// workspace (1024^3: 0.33 ms instead of 2.1).
constexpr int kCrossSlots = 2048;
constexpr int kCrossProbes = 16;

constexpr uint32_t kNoKey = 0xffffffffu;

// Inserts key into the block's set; false only when the set has no room
// for it (the caller then unites the pair itself).
__device__ __forceinline__ bool cross_insert(uint32_t *set, uint32_t key) {
  uint32_t h = (key * 0x9e3779b1u) >> (32 - 11);
#pragma unroll 1
  for (int probe = 0; probe < kCrossProbes; ++probe) {
    uint32_t cur = set[h];
    if (cur == key) return true;
    if (cur == kNoKey) {
      cur = atomicCAS(&set[h], kNoKey, key);
      if (cur == kNoKey || cur == key) return true;
    }
    h = (h + 1) & (kCrossSlots - 1);
  }
  return false;
}

// The two global ids a key stands for: the local root lv of tile t and the
// local root lu of the neighbour tile (bit k of nbr: one tile up along axis k).
__device__ __forceinline__ void cross_unite(const CGeo &g, const CTile &t,
                                            uint32_t key, int64_t *L) {
  const uint32_t lv = key & 0x1fffu, nbr = (key >> 13) & 7u, lu = key >> 16;
  const CTile tu{t.x0 + (nbr & 1u ? CTX : 0), t.y0 + (nbr & 2u ? CTY : 0),
                 t.z0 + (nbr & 4u ? CTZ : 0)};
  uf_unite_dev(L, ctile_global(g, t, (int)lv),
                    ctile_global(g, tu, (int)lu));
}

template <int B>
__global__ void __launch_bounds__(kCRows) k_cc_cross(CBatch<B> b) {
  static_assert(kCOwned <= (1 << 13), "13-bit local roots in the keys");
  // Rows (ly, lz) of the tile and one beyond in y and z: their words and first
  // run numbers in this x column of tiles, and in the next.
  constexpr int SY = CTY + 1, SN = SY * (CTZ + 1);
  __shared__ uint32_t w0[SN], wx[SN];
  __shared__ uint16_t b0[SN], bx[SN];
  __shared__ uint32_t set[kCrossSlots];
  const int r = threadIdx.x;
  for (int i = r; i < kCrossSlots; i += kCRows) set[i] = kNoKey;
  CGeo g;
  int64_t ti;
  const CGrid &d = cgrid_of(b, cc_tile_of_block(blockIdx.x, gridDim.x), &g,
                            &ti);
  int64_t *L = d.L;
  const CTile t = ctile_at(g, ti);
  const bool ux = t.x0 + CTX < g.X, uy = t.y0 + CTY < g.Y,
             uz = t.z0 + CTZ < g.Z;
  for (int i = r; i < SN; i += kCRows) {
    const int yy = i % SY, zz = i / SY;
    const bool oy = yy == CTY, oz = zz == CTZ;
    const bool in = (!oy || uy) && (!oz || uz);
    const int row = (oy ? 0 : yy) + CTY * (oz ? 0 : zz);
    const int64_t tn = in ? ti + (oy ? g.ntx : 0) + (oz ? g.ntx * g.nty : 0)
                          : ti;
    const CTileOut *o = ctile_out(d.loc, tn), *ox = ctile_out(d.loc, ux ? tn + 1 : tn);
    const uint32_t a = o->word[row], c = ox->word[row];
    const uint16_t ab = o->base[row], cb = ox->base[row];
    w0[i] = in ? a : 0u;
    b0[i] = ab;
    wx[i] = in && ux ? c : 0u;
    bx[i] = cb;
  }
  __syncthreads();
  const int y = r % CTY, z = r / CTY;
  const int i0 = y + SY * z, iy = i0 + 1, iz = i0 + SY, id = i0 + SY + 1;
  const uint32_t m = w0[i0];
  if (m) {
    const uint32_t st = run_starts(m), en = run_ends(m);
    const uint16_t *own = ctile_out(d.loc, ti)->root;
    const uint32_t nyr = y == CTY - 1 ? 2u : 0u, nzr = z == CTZ - 1 ? 4u : 0u;
    uint32_t last = kNoKey;
    // The run of x in this row with run k of the tile one up along `nbr`.
    auto pair = [&](int x, uint32_t nbr, uint32_t k) {
      const int64_t tn = ti + (nbr & 1u ? 1 : 0) + (nbr & 2u ? g.ntx : 0) +
                         (nbr & 4u ? g.ntx * g.nty : 0);
      const uint32_t lv = own[b0[i0] + run_of(st, x)];
      const uint32_t lu = ctile_out(d.loc, tn)->root[k];
      const uint32_t key = lv | (nbr << 13) | (lu << 16);
      if (key == last) return;  // a row's edges mostly repeat their roots
      last = key;
      if (!cross_insert(set, key)) cross_unite(g, t, key, L);
    };
    // Edges into row i of the tile up along `nbr`: x touches x and x+1 there,
    // so a run A = [a, b] touches B = [c, e] when they overlap (from max(a, c)
    // on) or c = b + 1.  `skip`: positions whose edges are implied.
    auto rows = [&](int i, uint32_t nbr, uint32_t skip) {
      const uint32_t nw = w0[i], sn = run_starts(nw);
      for (uint32_t c = m & nw & (st | sn) & ~skip; c; c &= c - 1) {
        const int x = __ffs((int)c) - 1;
        pair(x, nbr, b0[i] + run_of(sn, x));
      }
      for (uint32_t c = en & ~nw & (nw >> 1) & ~skip; c; c &= c - 1) {
        const int x = __ffs((int)c) - 1;  // at most CTX - 2
        pair(x, nbr, b0[i] + run_of(sn, x + 1));
      }
    };
    const uint32_t wy = w0[iy], wz = w0[iz];
    if (nyr) rows(iy, nyr, 0u);
    if (nzr) rows(iz, nzr, 0u);
    // An edge into the diagonal row is implied where x is masked in one of the
    // rows between.
    if (nyr | nzr) rows(id, nyr | nzr, wy | wz);
    // From the row's last vertex into the next tile in x: along x always; into
    // another row only when neither end has a masked neighbour on the way.
    constexpr int XL = CTX - 1;
    if (m >> XL) {
      const bool x0 = wx[i0] & 1u, xy = wx[iy] & 1u, xz = wx[iz] & 1u;
      if (x0) pair(XL, 1u, bx[i0]);
      if (xy && !x0 && !(wy >> XL)) pair(XL, 1u | nyr, bx[iy]);
      if (xz && !x0 && !(wz >> XL)) pair(XL, 1u | nzr, bx[iz]);
      if ((wx[id] & 1u) && !x0 && !xy && !xz && !((wy | wz | w0[id]) >> XL))
        pair(XL, 1u | nyr | nzr, bx[id]);
    }
  }
  // Each distinct triple once, spread over the block.
  __syncthreads();
  for (int i = r; i < kCrossSlots; i += kCRows) {
    const uint32_t key = set[i];
    if (key != kNoKey) cross_unite(g, t, key, L);
  }
}

// Every vertex's final label, plus `off` (a slab labelled inside a larger
// grid writes global ids).  The tile-local roots keep the unshifted root
// here, since concurrent walks read their entries as indices; k_cc_root_shift
// adds the offset to them afterwards.
// Each run's label is looked up once, into LDS; a vertex then needs its row's
// word and one LDS read.  Bound by the 8 bytes a vertex that are written
// (1024^3: 1.60 ms, 5.4 TB/s; 2.25 with a 16-bit root read for every vertex).
template <int B>
__global__ void __launch_bounds__(kCThreads) k_cc_final(CBatch<B> b) {
  __shared__ int64_t res[kCRuns];
  __shared__ uint32_t word[kCRows], base[kCRows];
  const int tid = threadIdx.x;
  CGeo g;
  int64_t ti;
  const CGrid &d = cgrid_of(b, cc_tile_of_block(blockIdx.x, gridDim.x), &g,
                            &ti);
  int64_t *L = d.L;
  const int64_t off = d.off;
  const CTile t = ctile_at(g, ti);
  const CTileOut *o = ctile_out(d.loc, ti);
  if (tid < kCRows) {
    word[tid] = o->word[tid];
    base[tid] = o->base[tid];
  }
  __syncthreads();
  const uint32_t runs =
      base[kCRows - 1] + (uint32_t)__popc(run_starts(word[kCRows - 1]));
  // Only tile-local roots are ever on a root path, and a root's entry is
  // overwritten (by its owner only) with its own final root, so concurrent
  // walks stay on ancestors and every entry ends as its final root.
  for (uint32_t i = tid; i < runs; i += kCThreads)
    res[i] = uf_root<int64_t>(L, ctile_global(g, t, o->root[i]));
  __syncthreads();
  const int cx = tid % CTX, cy = tid / CTX;
  const int64_t gx = t.x0 + cx, gy = t.y0 + cy;
  if (gx >= g.X || gy >= g.Y) return;
  const int nz = (int)((g.Z - t.z0) < CTZ ? (g.Z - t.z0) : CTZ);
  int64_t *const col = L + (gx + g.X * gy + g.XY * t.z0);
#pragma unroll 4
  for (int lz = 0; lz < nz; ++lz) {
    const int row = cy + CTY * lz;
    const uint32_t w = word[row], st = run_starts(w);
    int64_t v = -1;
    if ((w >> cx) & 1u) {
      const uint32_t k = base[row] + run_of(st, cx);
      v = res[k];
      // (a block-uniform test first)
      if (off && o->root[k] != row * CTX + cx) v += off;
    }
    __hip_atomic_store(col + g.XY * lz, v, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The tile-local roots' labels take the offset once no walk is in flight.
template <int B>
__global__ void __launch_bounds__(kCRows) k_cc_root_shift(CBatch<B> b) {
  const int r = threadIdx.x;
  CGeo g;
  int64_t ti;
  const CGrid &d = cgrid_of(b, cc_tile_of_block(blockIdx.x, gridDim.x), &g,
                            &ti);
  const CTile t = ctile_at(g, ti);
  const CTileOut *o = ctile_out(d.loc, ti);
  uint32_t i = o->base[r];
  for (uint32_t s = run_starts(o->word[r]); s; s &= s - 1, ++i) {
    const int l = r * CTX + __ffs((int)s) - 1;
    if (o->root[i] == l) d.L[ctile_global(g, t, l)] += d.off;
  }
}

// ---------------------------------------------------------------------------
// CSR graphs
// ---------------------------------------------------------------------------
//
// What bounds this path is random gathers, one per listed edge and pass: 50 to
// 60 G/s from an array that the last-level cache holds (256 MB), fewer from a
// larger one, and several times more from one that fits the L2s (4 MB each).
// So:
//  - the forest is 32-bit (n <= INT32_MAX) and lives in the upper half of the
//    labels, which a last pass widens in place: 200 MB instead of 400 for 50M
//    vertices;
//  - the mask is read as bits;
//  - most edges are settled before they are looked at one by one: every vertex
//    is hooked to its smallest masked neighbour among its first few (which
//    leaves a tree per local minimum of the ids, one vertex in fifteen of a
//    mesh), then rounds of single attempts to join two trees across a sampled
//    edge leave nearly everything of a large component in one; the tree that a
//    sample of the vertices names most often is marked in a bitmap, and the
//    pass over all edges gathers one bit for each edge of a marked vertex and
//    goes on only where a bit is clear.  (Sampling edges first and skipping the
//    most frequent component is the Afforest scheme of Sutton, Ben-Nun and
//    Barak, IPDPS 2018; the one-shot joins and the bitmap are this file's.)
// Every edge of every row is still examined, so rows that list an edge in one
// direction only are as good as symmetric ones.  50M vertices with 30 % in the
// mask take 5.7 ms instead of 14.2 (the union pass 2.7 instead of 8.9, the
// hooks 1.1 instead of 3.9, the joins 0.8), 1M vertices without a mask 0.25
// instead of 0.73.

// Edges of a CSR row handled together, so that their gathers overlap.
constexpr int kEdgeChunk = 8;

// Unions of v with u[j] for every j with need[j]: the roots of v and of
// those u[j] are found first with all the walks side by side (each step's
// loads for every walk issued before any is used; walks that are done, or not
// needed, reload v's own entry harmlessly, not a root's, where everyone's loads
// queue up: 1M vertices of a curve in no order 327 -> 290 us), then each u[j]'s
// root is hooked to v's in turn, the smaller root winning.  A hook whose root has
// moved meanwhile walks that pair again and retries; the merged root is then v's.
// (Hooking under any smaller member of the other tree, which spares reading its
// root, makes everyone's compare-and-swaps meet on the large tree's root instead:
// 100,000 vertices with 100,000 random edges 175 -> 234 us.)
__device__ __forceinline__ void uf_unite_row_dev(
    int32_t *par, int32_t v, const int32_t (&u)[kEdgeChunk],
    const bool (&need)[kEdgeChunk]) {
  constexpr int W = kEdgeChunk + 1;
  int32_t r[W];
  bool open[W];
  r[0] = v;
  open[0] = true;
#pragma unroll
  for (int j = 0; j < kEdgeChunk; ++j) {
    r[j + 1] = need[j] ? u[j] : v;
    open[j + 1] = need[j];
  }
  for (;;) {
    bool any = false;
#pragma unroll
    for (int i = 0; i < W; ++i) any |= open[i];
    if (!any) break;
    int32_t pr[W], gr[W];
#pragma unroll
    for (int i = 0; i < W; ++i) pr[i] = ld_dev(&par[open[i] ? r[i] : v]);
#pragma unroll
    for (int i = 0; i < W; ++i) gr[i] = ld_dev(&par[open[i] ? pr[i] : v]);
#pragma unroll
    for (int i = 0; i < W; ++i) {
      if (!open[i]) continue;
      if (pr[i] == r[i]) {
        open[i] = false;
      } else if (gr[i] == pr[i]) {
        r[i] = pr[i];
        open[i] = false;
      } else {
        __hip_atomic_store(&par[r[i]], gr[i], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        r[i] = gr[i];
      }
    }
  }
  int32_t rv = r[0];
#pragma unroll
  for (int j = 0; j < kEdgeChunk; ++j) {
    if (!need[j]) continue;
    int32_t a = rv, b = r[j + 1];
    for (;;) {
      if (a == b) {
        rv = a;
        break;
      }
      if (a > b) {
        const int32_t t = a;
        a = b;
        b = t;
      }
      int32_t expect = b;
      if (__hip_atomic_compare_exchange_strong(
              &par[b], &expect, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
              __HIP_MEMORY_SCOPE_AGENT)) {
        rv = a;
        break;
      }
      uf_find2_dev(par, a, b);  // b moved meanwhile; retry from the new trees
    }
  }
}

// Bit v of a bitmap over the vertices.
__device__ __forceinline__ bool bit_of(const uint32_t *bits, int32_t v) {
  return (bits[(uint32_t)v >> 5] >> ((uint32_t)v & 31u)) & 1u;
}

// One 64-bit word of a bitmap per wave of vertices.
__device__ __forceinline__ void put_bits(uint32_t *bits, int64_t v, bool on) {
  const unsigned long long m = __ballot(on);
  if ((threadIdx.x & 63) == 0)
    reinterpret_cast<unsigned long long *>(bits)[v >> 6] = m;
}

__global__ void __launch_bounds__(kBlock)
k_csr_mask_bits(int64_t n, const uint8_t *__restrict__ mask, uint32_t *bits) {
  const int64_t v = gid();
  const bool on = v < n && mask[v];
  if (((v | 63) - 63) < n) put_bits(bits, v, on);
}

// The graph as the passes see it; `bits` is the mask as a bitmap (or NULL, and
// the mask's bytes are read).
struct CsrGraph {
  int64_t n;
  const int64_t *rp;
  const int32_t *ci;
  const uint8_t *mask;
  const uint32_t *bits;
};

__device__ __forceinline__ bool csr_in(const CsrGraph &g, int32_t v) {
  return !g.mask || (g.bits ? bit_of(g.bits, v) : g.mask[v] != 0);
}

// A chunk of a row: the loads are unconditional, at indices kept in range (the
// chunk's first entry; the vertex itself), so that a chunk's loads of each
// kind are all issued before any is used.  Entries past the row, or out of
// range (reported in the result), become v.
__device__ __forceinline__ bool csr_chunk(const CsrGraph &g, int32_t v,
                                          int64_t e0, int64_t end,
                                          int32_t (&u)[kEdgeChunk]) {
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kEdgeChunk; ++j) u[j] = g.ci[e0 + j < end ? e0 + j : e0];
#pragma unroll
  for (int j = 0; j < kEdgeChunk; ++j) {
    const bool ok = u[j] >= 0 && (int64_t)u[j] < g.n;
    bad |= e0 + j < end && !ok;
    if (e0 + j >= end || !ok) u[j] = v;
  }
  return bad;
}

// Hook to the smallest masked vertex among v and the first chunk of its row.
__global__ void __launch_bounds__(kBlock)
k_csr_init(CsrGraph g, int32_t *__restrict__ P, unsigned long long *ctr) {
  const int64_t i = gid();
  if (i < kNumCounters) ctr[i] = 0ull;  // (grids are of whole blocks)
  if (i >= g.n) return;
  const int32_t v = (int32_t)i;
  int32_t best = -1;
  if (csr_in(g, v)) {
    best = v;
    const int64_t e0 = g.rp[i], end = g.rp[i + 1];
    if (e0 < end) {
      int32_t u[kEdgeChunk];
      bool in[kEdgeChunk];
      (void)csr_chunk(g, v, e0, end, u);
#pragma unroll
      for (int j = 0; j < kEdgeChunk; ++j) in[j] = csr_in(g, u[j]);
#pragma unroll
      for (int j = 0; j < kEdgeChunk; ++j)
        if (in[j] && u[j] < best) best = u[j];
    }
  }
  P[i] = best;
}

// Root of x if it is at most kLeg steps away, else -1 (the walk may grow as fast
// as it goes on: other threads hook the roots that it reaches).
constexpr int kLeg = 32;

__device__ __forceinline__ int32_t uf_root_near(const int32_t *P, int32_t x) {
#pragma unroll 1
  for (int k = 0; k < kLeg; ++k) {
    const int32_t p = __hip_atomic_load(&P[x], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
    if (p == x) return x;
    x = p;
  }
  return -1;
}

// One attempt to join v's tree with that of one entry of its row, for one in
// `stride` waves of vertices: the larger root is hooked if it still is a root.
// Another thread may have hooked it first, or the roots may have moved far; later
// rounds and the pass over all edges make good what is left then, where retrying
// until the trees are one has a million threads queue up on a handful of roots
// (1.5 ms), and walking on along a curve with rising ids, where the hooks form
// one chain, takes up to 20 ms for 1M vertices.
__device__ __forceinline__ void csr_join(const CsrGraph &g, int32_t *P,
                                         int64_t i, int pick) {
  if (i >= g.n) return;
  int32_t a = P[i];
  if (a < 0) return;
  const int64_t e0 = g.rp[i], deg = g.rp[i + 1] - e0;
  if (deg <= 0) return;
  const int32_t u = g.ci[e0 + (pick < deg ? deg - 1 - pick : 0)];
  if (u < 0 || (int64_t)u >= g.n) return;
  int32_t b = P[u];
  if (b < 0 || a == b) return;
  a = uf_root_near(P, a);
  b = uf_root_near(P, b);
  if (a == b || a < 0 || b < 0) return;
  const int32_t lo = a < b ? a : b;
  int32_t hi = a < b ? b : a;
  if (ld_dev(&P[hi]) == hi)
    __hip_atomic_compare_exchange_strong(&P[hi], &hi, lo, __ATOMIC_RELAXED,
                                         __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(kBlock)
k_csr_join(CsrGraph g, int32_t *P, int stride, int pick) {
  csr_join(g, P, (gid() >> 6) * stride * 64 + (threadIdx.x & 63), pick);
}

// The rounds after the first in one launch, for graphs where a launch costs more
// than the order of the rounds is worth.
template <int S1, int S2, int S3>
__global__ void __launch_bounds__(kBlock)
k_csr_join_rest(CsrGraph g, int32_t *P) {
  const int64_t w = gid() >> 6;
  const int64_t i = w * S1 * 64 + (threadIdx.x & 63);
  csr_join(g, P, i, 1);
  if (w % (S2 / S1) == 0) csr_join(g, P, i, 2);
  if (w % (S3 / S1) == 0) csr_join(g, P, i, 3);
}

// Every vertex straight to its root.  Most trees are shallow, but hooks and
// joins can also leave a chain through half the vertices (ids that rise along a
// curve).  So a walk that has not ended after kLeg steps writes how far it has
// come into its own entry, which nobody else writes, and goes on with loads that
// see what the others have written: a leg then steps over all that the leg
// before covered (the vertices below, whose threads started earlier, do the
// same).
__device__ __forceinline__ int32_t csr_settle(int32_t *P, int64_t v) {
  int32_t x = __hip_atomic_load(&P[v], __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
  bool open = x >= 0;
#pragma unroll 1
  for (int k = 0; open && k < kLeg; ++k) {
    const int32_t p = __hip_atomic_load(&P[x], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
    open = p != x;
    x = p;
  }
  while (open) {
    __hip_atomic_store(&P[v], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 1
    for (int k = 0; open && k < kLeg; ++k) {
      const int32_t p = ld_dev(&P[x]);
      open = p != x;
      x = p;
    }
  }
  return x;
}

__global__ void __launch_bounds__(kBlock)
k_csr_compress(int64_t n, int32_t *P) {
  const int64_t v = gid();
  if (v >= n) return;
  const int32_t x = csr_settle(P, v);
  if (x >= 0)
    __hip_atomic_store(&P[v], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The last compression: labels below `half`, which lie below the forest, are
// written at once.
__global__ void __launch_bounds__(kBlock)
k_csr_final(int64_t n, int64_t half, int32_t *P, int64_t *L) {
  const int64_t v = gid();
  if (v >= n) return;
  const int32_t x = csr_settle(P, v);
  if (v < half)
    L[v] = (int64_t)x;
  else if (x >= 0)
    __hip_atomic_store(&P[v], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The root that a sample of the vertices names most often (-2: none is in the
// mask), found by a block of T threads; a guess, which only speed depends on.
template <int T, int SAMPLE>
__device__ __forceinline__ int32_t csr_giant(int64_t n,
                                             const int32_t *__restrict__ P) {
  constexpr int SLOTS = 2 * SAMPLE, LOG = __builtin_ctz(SLOTS);
  __shared__ int32_t key[SLOTS];
  __shared__ uint32_t cnt[SLOTS];
  __shared__ unsigned long long best;
  for (int i = threadIdx.x; i < SLOTS; i += T) {
    key[i] = -1;
    cnt[i] = 0;
  }
  if (threadIdx.x == 0) best = 0;
  __syncthreads();
  for (int k = threadIdx.x; k < SAMPLE; k += T) {
    const int32_t r =
        P[(uint64_t)((uint32_t)k * 0x9e3779b1u) * (uint64_t)n >> 32];
    if (r < 0) continue;
    uint32_t h = ((uint32_t)r * 0x85ebca6bu) >> (32 - LOG);
    for (;;) {  // half the slots stay empty
      const int32_t cur = atomicCAS(&key[h], -1, r);
      if (cur == -1 || cur == r) break;
      h = (h + 1) & (SLOTS - 1);
    }
    atomicAdd(&cnt[h], 1u);
  }
  __syncthreads();
  unsigned long long top = 0;
  for (int i = threadIdx.x; i < SLOTS; i += T)
    if (cnt[i]) {
      const unsigned long long c =
          (unsigned long long)cnt[i] << 32 | (uint32_t)key[i];
      top = c > top ? c : top;
    }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long c = __shfl_xor(top, o);
    top = c > top ? c : top;
  }
  if ((threadIdx.x & 63) == 0 && top) atomicMax(&best, top);
  __syncthreads();
  return best ? (int32_t)(uint32_t)best : -2;
}

__global__ void __launch_bounds__(1024)
k_csr_giant(int64_t n, const int32_t *__restrict__ P, int32_t *giant) {
  const int32_t r = csr_giant<1024, 2048>(n, P);
  if (threadIdx.x == 0) *giant = r;
}

// The tree's vertices as a bitmap: from the root that k_csr_giant has found, or
// (in graphs where a launch costs more) that every block finds for itself.
__global__ void __launch_bounds__(kBlock)
k_csr_mark_small(int64_t n, const int32_t *__restrict__ P, uint32_t *bits) {
  const int32_t r = csr_giant<kBlock, 512>(n, P);
  const int64_t v = gid();
  const bool on = v < n && P[v] == r;
  if (((v | 63) - 63) < n) put_bits(bits, v, on);
}

__global__ void __launch_bounds__(kBlock)
k_csr_giant_bits(int64_t n, const int32_t *__restrict__ P,
                 const int32_t *__restrict__ giant, uint32_t *bits) {
  const int64_t v = gid();
  const bool on = v < n && P[v] == *giant;
  if (((v | 63) - 63) < n) put_bits(bits, v, on);
}

// One union per listed edge between two masked vertices, where none of the
// cheaper looks settles it: both ends in the marked tree (two bits), then
// equal entries (cached reads: an old value is still an ancestor, so equal
// values prove the two are connected).  Checks every index.
__global__ void __launch_bounds__(kBlock)
k_csr_union(CsrGraph g, int32_t *P, const uint32_t *__restrict__ marked,
            unsigned long long *ctr) {
  const int64_t i = gid();
  bool bad = false;
  const int32_t v = (int32_t)i;
  const int32_t pv =
      i < g.n ? __hip_atomic_load(&P[i], __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP)
              : -1;
  if (pv >= 0) {
    const int64_t e1 = g.rp[i], end = g.rp[i + 1];
    bool open = true;
    if (marked && bit_of(marked, v)) {
      // A bit per edge, sixteen at a time: most rows end here.
      constexpr int K = 2 * kEdgeChunk;
      uint32_t all = 1u;
      for (int64_t e0 = e1; e0 < end; e0 += K) {
        int32_t u[K];
        uint32_t w[K];
#pragma unroll
        for (int j = 0; j < K; ++j) u[j] = g.ci[e0 + j < end ? e0 + j : e0];
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const bool ok = u[j] >= 0 && (int64_t)u[j] < g.n;
          bad |= !ok;
          u[j] = ok ? u[j] : v;
        }
#pragma unroll
        for (int j = 0; j < K; ++j) w[j] = marked[(uint32_t)u[j] >> 5];
#pragma unroll
        for (int j = 0; j < K; ++j) all &= w[j] >> ((uint32_t)u[j] & 31u);
      }
      open = !all;
    }
    for (int64_t e0 = e1; open && e0 < end; e0 += kEdgeChunk) {
      int32_t u[kEdgeChunk], pu[kEdgeChunk];
      bool need[kEdgeChunk];
      bad |= csr_chunk(g, v, e0, end, u);
#pragma unroll
      for (int j = 0; j < kEdgeChunk; ++j)
        pu[j] = __hip_atomic_load(&P[u[j]], __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
      bool any = false;
#pragma unroll
      for (int j = 0; j < kEdgeChunk; ++j) {
        need[j] = u[j] != v && pu[j] >= 0 && pu[j] != pv;  // masked, elsewhere
        any |= need[j];
      }
      if (any) uf_unite_row_dev(P, v, u, need);
    }
  }
  flag_any(bad, ctr + kCtrBadIndex);
}

// The labels of [a, b) from the forest in the labels' upper half (32-bit words
// n and up).  Label v takes words 2v and 2v + 1, so with b <= (n + a) / 2 no
// entry is overwritten before it is read.
__global__ void __launch_bounds__(kBlock)
k_csr_widen(int64_t a, int64_t b, const int32_t *P, int64_t *L) {
  const int64_t v = a + gid();
  if (v < b) L[v] = (int64_t)P[v];
}

// The last stretch [a, n), at most kTail vertices, in one block: every entry
// is read before any label is written.  `walk`: the entries are not roots yet
// (a = 0; nothing is overwritten while the block walks).  The call's last kernel:
// it also hands the counters to the host, where a copy would take longer.
constexpr int kTail = 16384;

__global__ void __launch_bounds__(1024)
k_csr_widen_tail(int64_t a, int64_t n, bool walk, const int32_t *P,
                 int64_t *L, const unsigned long long *ctr,
                 unsigned long long *hctr) {
  constexpr int K = kTail / 1024;
  if (threadIdx.x < kNumCounters)
    __hip_atomic_store(hctr + threadIdx.x, ctr[threadIdx.x], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  int32_t r[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t v = a + threadIdx.x + k * 1024;
    r[k] = v < n ? P[v] : -1;
    if (walk && r[k] >= 0) r[k] = uf_root<int32_t>(P, (int32_t)v);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t v = a + threadIdx.x + k * 1024;
    if (v < n) L[v] = (int64_t)r[k];
  }
}

// ---------------------------------------------------------------------------
// Pointer forests
// ---------------------------------------------------------------------------

// One in-place jumping round; negative entries are not part of the forest.
__global__ void __launch_bounds__(kBlock)
k_jump64(int64_t *L, int64_t n, unsigned long long *ctr) {
  int64_t v = gid();
  bool changed = false;
  if (v < n) {
    int64_t u = L[v];
    if (u >= 0 && u != v) {
      int64_t w = __atomic_load_n(&L[u], __ATOMIC_RELAXED);
      if (w != u) {
        L[v] = w;
        changed = true;
      }
    }
  }
  flag_any(changed, ctr + kCtrChanged);
}

// Synchronous doubling: out[v] = in[in[v]].
__global__ void __launch_bounds__(kBlock)
k_double64(const int64_t *__restrict__ in, int64_t *__restrict__ out,
           int64_t n, unsigned long long *ctr) {
  int64_t v = gid();
  bool changed = false;
  if (v < n) {
    int64_t u = in[v];
    int64_t w = in[u];
    out[v] = w;
    changed = w != u;
  }
  flag_any(changed, ctr + kCtrChanged);
}

// Every pointer must be an id in [0, n) before any kernel follows it.
__global__ void __launch_bounds__(kBlock)
k_check_range(const int64_t *__restrict__ d, int64_t n,
              unsigned long long *ctr) {
  int64_t v = gid();
  flag_any(v < n && (d[v] < 0 || d[v] >= n), ctr + kCtrBadIndex);
}

int clear_changed(msc_ctx *ctx, hipStream_t s) {
  return zero_u64(ctx->dctr + kCtrChanged, 1, s);
}

// In-place doubling needs at most about log2(longest path) + 1 rounds; more
// than this many means the pointers hold a cycle (not a forest).
constexpr int kMaxRounds = 96;

}  // namespace

namespace {

// Masks per launch of a batched call: their descriptors travel as kernel
// arguments (64 bytes each).
constexpr int kCCBatch = 32;

// The grid-CC kernels over `nb` tiles of the masks in `b`.
template <int B>
int cc_launch(msc_ctx *ctx, const CBatch<B> &b, uint32_t nb, int64_t nverts,
              bool shift, hipStream_t s) {
  MSC_PHASE(ctx, s, "cc_tile", 3.0 * nverts,
            (k_cc_tile<B><<<nb, kCTileThreads, 0, s>>>(b)));
  MSC_PHASE(ctx, s, "cc_cross", 0.5 * nverts,
            (k_cc_cross<B><<<nb, kCRows, 0, s>>>(b)));
  MSC_PHASE(ctx, s, "cc_final", 10.0 * nverts,
            (k_cc_final<B><<<nb, kCThreads, 0, s>>>(b)));
  if (shift)
    MSC_PHASE(ctx, s, "cc_root_shift", 2.0 * nverts,
              (k_cc_root_shift<B><<<nb, kCRows, 0, s>>>(b)));
  return MSC_OK;
}

int64_t cc_tiles(int64_t X, int64_t Y, int64_t Z) {
  return ((X + CTX - 1) / CTX) * ((Y + CTY - 1) / CTY) * ((Z + CTZ - 1) / CTZ);
}

}  // namespace

size_t cc_grid_workspace(int n, const msc_mask *masks) {
  size_t need = 4096;
  for (int i = 0; i < n; ++i)
    need += align256((size_t)cc_tiles(masks[i].dims[0], masks[i].dims[1],
                                      masks[i].dims[2]) *
                     kCOwned * sizeof(uint16_t));
  return need;
}

int cc_grid_run(msc_ctx *ctx, const uint8_t *mask, int64_t X, int64_t Y,
                int64_t Z, int64_t *labels, hipStream_t s, bool sync,
                int64_t label_off) {
  const int64_t N = X * Y * Z;
  const int64_t ntiles = cc_tiles(X, Y, Z);
  if (ntiles > INT32_MAX) return MSC_ERANGE;
  MSC_TRY(reserve(ctx, ctx->ws,
                  align256(ntiles * kCOwned * sizeof(uint16_t)) + 4096));
  Carver cv(ctx->ws);
  uint16_t *loc = cv.take<uint16_t>(ntiles * kCOwned);
  CBatch<1> b{1, {CGrid{mask, labels, loc, label_off, X, Y, Z, 0u}}};
  MSC_TRY(cc_launch(ctx, b, (uint32_t)ntiles, N, label_off != 0, s));
  if (!sync) return MSC_OK;
  // Nothing to read back: the labels are the whole result.
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = N;
  ctx->stats.tile_x = CTX;
  ctx->stats.tile_y = CTY;
  ctx->stats.tile_z = CTZ;
  return MSC_OK;
}

int cc_grid_batch_run(msc_ctx *ctx, int n, const msc_mask *masks,
                      hipStream_t s) {
  int64_t total = 0;
  for (int i = 0; i < n; ++i) {
    const int64_t *d = masks[i].dims;
    if (cc_tiles(d[0], d[1], d[2]) > INT32_MAX) return MSC_ERANGE;
    total += d[0] * d[1] * d[2];
  }
  MSC_TRY(reserve(ctx, ctx->ws, cc_grid_workspace(n, masks)));
  Carver cv(ctx->ws);
  CBatch<kCCBatch> b{};
  uint64_t tiles = 0;
  int64_t verts = 0;
  for (int i = 0; i <= n; ++i) {
    const int64_t *d = i < n ? masks[i].dims : nullptr;
    const int64_t nt = d ? cc_tiles(d[0], d[1], d[2]) : 0;
    // Launch what is collected when the batch is full, would pass 2^31 - 1
    // tiles, or the masks are exhausted.
    if (b.n > 0 && (i == n || b.n == kCCBatch || tiles + nt > INT32_MAX)) {
      MSC_TRY(cc_launch(ctx, b, (uint32_t)tiles, verts, false, s));
      b.n = 0;
      tiles = 0;
      verts = 0;
    }
    if (i == n) break;
    const int64_t N = d[0] * d[1] * d[2];
    b.g[b.n++] = CGrid{masks[i].mask, masks[i].labels,
                       cv.take<uint16_t>(nt * kCOwned), 0, d[0], d[1], d[2],
                       (uint32_t)tiles};
    tiles += (uint64_t)nt;
    verts += N;
  }
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = total;
  ctx->stats.tile_x = CTX;
  ctx->stats.tile_y = CTY;
  ctx->stats.tile_z = CTZ;
  return MSC_OK;
}

// Graphs from this size on take the steps that settle most edges early (8,000
// vertices of a mesh, ids in no order: 64 us with them, 122 without; 1,728: 81
// and 75, as each step is a launch.  Where rows are short or ids lie in order the
// launches are all that they add up to 128k vertices: 16k of a curve 104 us and
// 80, 8,000 of a mesh in grid order 63 and 53; the entry count that would tell
// is on the device).
constexpr int64_t kCsrLarge = 1 << 12;
// Rounds of joins, each over one in so many waves of vertices: trees are fewer
// and larger from round to round, so fewer attempts reach all of them.  With
// every vertex in each of four rounds 50M vertices take 8.4 ms instead of 7.1,
// 1M take 0.29 instead of 0.25; with two rounds too many trees are left and
// 1M take 1.7 ms.  Half as many attempts in every round do from kJoinHalf
// vertices on (50M: 7.0 -> 6.3 ms, 8M: 1.44 -> 1.31; 1M: 0.25 and 0.26, and
// 8,000 take 108 us instead of 83).
constexpr int kJoinStride[] = {1, 4, 16, 32};
constexpr int64_t kJoinHalf = 1 << 21;
constexpr int kJoins = sizeof(kJoinStride) / sizeof(int);
// Up to so many vertices the rounds after the first share a launch (mesh of 20^3:
// 71 -> 60 us, 10,000 vertices and random edges 97 -> 91), and the tree to mark
// is found by every block for itself (curve of 64k vertices 115 -> 106).  Rounds
// in one launch see less of each other's joins: 100,000 vertices with 200,000
// random entries take 276 us so, 144 in launches of their own.
constexpr int64_t kJoinFused = 1 << 14, kMarkFused = 1 << 17;

int cc_csr_run(msc_ctx *ctx, int64_t n, const int64_t *row_ptr,
               const int32_t *col_idx, const uint8_t *mask, int64_t *labels,
               hipStream_t s) {
  // The labels' own memory holds everything: the forest in the upper half, the
  // bitmaps (n / 8 bytes each) in the lower.
  int32_t *P = reinterpret_cast<int32_t *>(labels) + n;
  const bool large = n >= kCsrLarge;
  const int64_t words = (n + 63) / 64 * 2;
  uint32_t *mbits = reinterpret_cast<uint32_t *>(labels);
  uint32_t *marked = large ? mbits + words : nullptr;
  const unsigned nb = grid_for(n);
  CsrGraph g{n, row_ptr, col_idx, mask, nullptr};
  int32_t *giant = reinterpret_cast<int32_t *>(ctx->dctr + kCtrGiant);
  if (large && mask) {
    g.bits = mbits;
    k_csr_mask_bits<<<nb, kBlock, 0, s>>>(n, mask, mbits);
  }
  MSC_PHASE(ctx, s, "csr_init", 17.0 * n,
            (k_csr_init<<<nb, kBlock, 0, s>>>(g, P, ctx->dctr)));
  MSC_PHASE(ctx, s, "csr_compress", 8.0 * n,
            (k_csr_compress<<<nb, kBlock, 0, s>>>(n, P)));
  if (large) {
    const bool fused = n <= kJoinFused;
    for (int k = 0; k < (fused ? 1 : kJoins); ++k) {
      const int stride = kJoinStride[k] * (n >= kJoinHalf ? 2 : 1);
      const int64_t waves = (n + 64 * stride - 1) / (64 * stride);
      MSC_PHASE(ctx, s, "csr_join", 21.0 * n,
                (k_csr_join<<<grid_for(64 * waves), kBlock, 0, s>>>(g, P,
                                                                    stride, k)));
      if (k == 0) k_csr_compress<<<nb, kBlock, 0, s>>>(n, P);
    }
    static_assert(kJoins == 4, "the rounds of k_csr_join_rest");
    if (fused)
      MSC_PHASE(ctx, s, "csr_join", 21.0 * n,
                (k_csr_join_rest<kJoinStride[1], kJoinStride[2], kJoinStride[3]>
                 <<<grid_for((n + 64 * kJoinStride[1] - 1) /
                             (64 * kJoinStride[1]) * 64),
                    kBlock, 0, s>>>(g, P)));
    k_csr_compress<<<nb, kBlock, 0, s>>>(n, P);
    if (n <= kMarkFused)
      MSC_PHASE(ctx, s, "csr_mark", 4.0 * n,
                (k_csr_mark_small<<<nb, kBlock, 0, s>>>(n, P, marked)));
    else
      MSC_PHASE(ctx, s, "csr_mark", 4.0 * n,
                (k_csr_giant<<<1, 1024, 0, s>>>(n, P, giant),
                 k_csr_giant_bits<<<nb, kBlock, 0, s>>>(n, P, giant, marked)));
  }
  MSC_PHASE(ctx, s, "csr_union", 13.0 * n,
            (k_csr_union<<<nb, kBlock, 0, s>>>(g, P, marked, ctx->dctr)));
  int64_t a = 0;
  if (n > kTail) {
    MSC_PHASE(ctx, s, "csr_final", 8.0 * n,
              (k_csr_final<<<nb, kBlock, 0, s>>>(n, n / 2, P, labels)));
    a = n / 2;
    while (n - a > kTail) {
      const int64_t b = (n + a) / 2;
      k_csr_widen<<<grid_for(b - a), kBlock, 0, s>>>(a, b, P, labels);
      a = b;
    }
  }
  k_csr_widen_tail<<<1, 1024, 0, s>>>(a, n, a == 0, P, labels, ctx->dctr,
                                      ctx->dhctr);
  MSC_HIP_TRY(hipGetLastError());
  MSC_HIP_TRY(hipStreamSynchronize(s));
  if (ctx->prof.on) ctx->prof.flush();
  if (ctx->hctr[kCtrBadIndex]) return MSC_EINVAL;
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = n;
  return MSC_OK;
}

int jump_run(msc_ctx *ctx, int64_t *d, int64_t n, int rounds, int sync,
             hipStream_t s) {
  MSC_TRY(clear_counters(ctx, s));
  MSC_PHASE(ctx, s, "check_range", 8.0 * n,
            (k_check_range<<<grid_for(n), kBlock, 0, s>>>(d, n, ctx->dctr)));
  MSC_TRY(read_counters(ctx, s));
  if (ctx->hctr[kCtrBadIndex]) return MSC_EINVAL;
  if (!sync) {
    for (int r = 0; rounds == 0 || r < rounds; ++r) {
      if (rounds == 0 && r == kMaxRounds) return MSC_EINVAL;
      MSC_TRY(clear_changed(ctx, s));
      MSC_PHASE(ctx, s, "jump64_round", 24.0 * n,
                (k_jump64<<<grid_for(n), kBlock, 0, s>>>(d, n, ctx->dctr)));
      if (rounds == 0) {
        MSC_TRY(read_counters(ctx, s));
        if (!ctx->hctr[kCtrChanged]) break;
      }
    }
    return MSC_OK;
  }
  MSC_TRY(reserve(ctx, ctx->ws, align256(n * sizeof(int64_t)) + 4096));
  Carver cv(ctx->ws);
  int64_t *tmp = cv.take<int64_t>(n);
  int64_t *src = d, *dst = tmp;
  for (int r = 0; rounds == 0 || r < rounds; ++r) {
    if (rounds == 0 && r == kMaxRounds) return MSC_EINVAL;
    MSC_TRY(clear_changed(ctx, s));
    MSC_PHASE(ctx, s, "double64_round", 24.0 * n,
              (k_double64<<<grid_for(n), kBlock, 0, s>>>(src, dst, n,
                                                         ctx->dctr)));
    int64_t *t = src;
    src = dst;
    dst = t;
    if (rounds == 0) {
      MSC_TRY(read_counters(ctx, s));
      if (!ctx->hctr[kCtrChanged]) break;
    }
  }
  if (src != d)
    MSC_HIP_TRY(hipMemcpyAsync(d, src, n * sizeof(int64_t),
                               hipMemcpyDeviceToDevice, s));
  return MSC_OK;
}

// ---------------------------------------------------------------------------
// Grid CC with no allocation (for callers that cannot allocate: code under
// graph capture, tight serving loops).  The tiles' slots live in one static
// device array per GPU, taken once per device by symbol address.
// ---------------------------------------------------------------------------

namespace {

// A slot of 2^13 16-bit words per tile (see CTileOut): 2^27 words (256 MiB per
// GPU the library runs on, held until the process ends) bound a call at 2^14
// tiles of 32x16x16 (512^3 vertices).
constexpr int64_t kNoAllocEntries = INT64_C(1) << 27;
static __device__ __align__(256) uint16_t scratch[kNoAllocEntries];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint16_t *g_scratch_ptr[kMaxDevices] = {};

// The array's device address on `dev`, the current device (the host-side
// name `scratch` is only a stand-in, never a device address).
int scratch_of(int dev, uint16_t **out) {
  if (dev < 0 || dev >= kMaxDevices) return MSC_EINVAL;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return MSC_EHIP;
    }
    g_scratch_ptr[dev] = static_cast<uint16_t *>(p);
  }
  *out = g_scratch_ptr[dev];
  return MSC_OK;
}

}  // namespace
}  // namespace msc

extern "C" int cc_label_grid_noalloc(const uint8_t *mask,
                                     const int64_t dims[3], int64_t *labels,
                                     void *stream) {
  using namespace msc;
  if (!mask || !labels || !dims) return MSC_EINVAL;
  for (int k = 0; k < 3; ++k)
    if (dims[k] < 1) return MSC_EINVAL;
  // Each factor is bounded first, so that the tile count cannot overflow.
  if (dims[0] > kNoAllocEntries || dims[1] > kNoAllocEntries ||
      dims[2] > kNoAllocEntries ||
      cc_tiles(dims[0], dims[1], dims[2]) * kCOwned > kNoAllocEntries)
    return MSC_ERANGE;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return MSC_EHIP;
  uint16_t *loc = nullptr;
  MSC_TRY(scratch_of(dev, &loc));
  const int64_t X = dims[0], Y = dims[1], Z = dims[2];
  const unsigned nb = (unsigned)cc_tiles(X, Y, Z);
  const CBatch<1> b{1, {CGrid{mask, labels, loc, 0, X, Y, Z, 0u}}};
  hipStream_t s = static_cast<hipStream_t>(stream);
  // Everything of a tile's slot that the kernels read k_cc_tile writes first
  // (all rows, and the runs that they hold), so nothing is cleared.
  k_cc_tile<1><<<nb, kCTileThreads, 0, s>>>(b);
  k_cc_cross<1><<<nb, kCRows, 0, s>>>(b);
  k_cc_final<1><<<nb, kCThreads, 0, s>>>(b);
  return hipGetLastError() == hipSuccess ? MSC_OK : MSC_EHIP;
}

namespace msc {

// ---------------------------------------------------------------------------
// Virtual ranks: slab-local labelling, then the exchange across slab
// boundaries (Alg. 3 with the distributed phase it shares with the MS
// segmentation).  Slab r holds planes [r*Z/R, (r+1)*Z/R).
// ---------------------------------------------------------------------------

namespace {

// A slab's labels name vertices by their id within the slab; adding the id
// of the slab's first vertex makes them global ids.
// The exchange at the boundary between plane zb (top of one slab) and
// zb + 1 (bottom of the next): every Freudenthal edge that crosses it,
// (x, y, zb) -- (x + dx, y + dy, zb + 1) for dx, dy in {0, 1}, joins the
// two endpoints' trees when both are in the mask.  L is the parent array:
// every label is a root of its slab's forest, and the smaller root wins.
// All R - 1 boundaries in one launch (grid y strides over them): unions are
// safe to run concurrently, and the boundaries' latency-bound root walks
// overlap.
__global__ void __launch_bounds__(kBlock)
k_rank_cc_stitch(const uint8_t *__restrict__ mask, int64_t X, int64_t Y,
                 int64_t Z, int64_t R, int64_t *L) {
  const int64_t XY = X * Y;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool in = i < XY;
  const int64_t x = in ? i % X : 0, y = in ? i / X : 0;
  for (int64_t r = 1 + blockIdx.y; r < R; r += gridDim.y) {
    const int64_t zb = r * Z / R - 1;
    const int64_t u = i + XY * zb;
    const bool mu = in && mask[u];
    // The slab labels of both ends, joined once per distinct pair in a run
    // of lanes: neighbouring vertices mostly carry the same two labels, and
    // letting every lane unite them would pile compare-and-swaps onto the
    // same root.
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int dx = e & 1, dy = e >> 1;
      int64_t a = -1, b = -1;
      if (mu && x + dx < X && y + dy < Y) {
        const int64_t w = u + XY + dx + X * dy;
        if (mask[w]) {
          a = L[u];
          b = L[w];
        }
      }
      const int64_t pa = __shfl_up(a, 1), pb = __shfl_up(b, 1);
      const bool first = (threadIdx.x & 63) == 0 || pa != a || pb != b;
      if (a >= 0 && a != b && first) uf_unite_dev(L, a, b);
    }
  }
}

// Every masked vertex takes the root of its label (the smallest id of its
// component); run once no union is in flight.
__global__ void __launch_bounds__(kBlock)
k_rank_cc_final(int64_t *L, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) {
    const int64_t v = L[i];
    if (v >= 0) L[i] = uf_root<int64_t>(L, v);
  }
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

int cc_grid_ranks_run(msc_ctx *ctx, const uint8_t *mask, int64_t X,
                      int64_t Y, int64_t Z, int ranks, int64_t *labels,
                      hipStream_t s) {
  const int64_t XY = X * Y, N = XY * Z;
  // Room for the thickest slab's tiles: no slab grows the workspace while the
  // kernels of the ones before it are queued on it.
  const msc_mask thickest{mask, {X, Y, (Z + ranks - 1) / ranks}, labels};
  MSC_TRY(reserve(ctx, ctx->ws, cc_grid_workspace(1, &thickest)));
  for (int r = 0; r < ranks; ++r) {
    const int64_t z0 = r * Z / ranks, z1 = (r + 1) * Z / ranks;
    // No host round trip per slab: the slabs queue on the stream (the
    // tile-local workspace is sized for the largest slab up front).
    // Each slab is labelled in place with global ids (its first id as the
    // label offset).
    MSC_TRY(cc_grid_run(ctx, mask + XY * z0, X, Y, z1 - z0, labels + XY * z0,
                        s, false, XY * z0));
  }
  if (ranks > 1) {
    const unsigned by = ranks - 1 < 65535 ? (unsigned)(ranks - 1) : 65535u;
    MSC_PHASE(ctx, s, "rank_cc_stitch", 2.0 * XY * (ranks - 1),
              (k_rank_cc_stitch<<<dim3(blocks_for(XY), by), kBlock, 0, s>>>(
                  mask, X, Y, Z, ranks, labels)));
  }
  if (ranks > 1)
    MSC_PHASE(ctx, s, "rank_cc_final", 16.0 * N,
              (k_rank_cc_final<<<blocks_for(N), kBlock, 0, s>>>(labels, N)));
  MSC_TRY(read_counters(ctx, s));
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = N;
  return MSC_OK;
}

// ---------------------------------------------------------------------------
// CSR adjacency of a tetrahedral complex (the mesh of the explicit pipeline
// and of msc_segment_csr): every tetrahedron's vertices are neighbours of
// one another.  Per vertex: candidates gathered from its tetrahedra (once per
// block of tetrahedra that holds the edge), then the distinct ones written in
// increasing order.  No global sort: vertex degrees are small, so each row is
// deduplicated and ranked by comparing its candidates with one another.
// ---------------------------------------------------------------------------

namespace {

constexpr int kScan = 1024;

// Exclusive prefix of x over the block (1024 threads) and the block total.
__device__ __forceinline__ uint64_t block_scan64(uint64_t x, uint64_t *tmp,
                                                 uint64_t *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t inc = x;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) tmp[w] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t run = 0;
    for (int k = 0; k < kScan / 64; ++k) {
      const uint64_t t = tmp[k];
      tmp[k] = run;
      run += t;
    }
    tmp[kScan / 64] = run;
  }
  __syncthreads();
  const uint64_t ex = inc - x + tmp[w];
  *total = tmp[kScan / 64];
  __syncthreads();
  return ex;
}

__global__ void __launch_bounds__(kScan)
k_scan64_blocks(const uint32_t *__restrict__ cnt, int64_t n, int64_t *out,
                uint64_t *bsum) {
  __shared__ uint64_t tmp[kScan / 64 + 1];
  const int64_t i = (int64_t)blockIdx.x * kScan + threadIdx.x;
  uint64_t tot = 0;
  const uint64_t ex = block_scan64(i < n ? cnt[i] : 0u, tmp, &tot);
  if (i < n) out[i] = (int64_t)ex;
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Block totals to block offsets in place (one block); the grand total goes
// to out[n].
__global__ void __launch_bounds__(kScan)
k_scan64_sums(uint64_t *bsum, int64_t nb, int64_t *out, int64_t n) {
  __shared__ uint64_t tmp[kScan / 64 + 1];
  uint64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kScan) {
    const int64_t i = b0 + threadIdx.x;
    uint64_t tot = 0;
    const uint64_t ex = block_scan64(i < nb ? bsum[i] : 0u, tmp, &tot);
    if (i < nb) bsum[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) out[n] = (int64_t)carry;
}

__global__ void __launch_bounds__(kBlock)
k_scan64_add(int64_t *out, int64_t n, const uint64_t *__restrict__ bsum) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) out[i] += (int64_t)bsum[i / kScan];
}

__global__ void __launch_bounds__(kBlock)
k_zero32(uint32_t *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = 0;
}

// A block takes kTets tetrahedra and reduces them in LDS before it touches
// device memory: an open-addressed table of their distinct vertices, and one
// of their distinct edges (pairs of vertex slots).  Tetrahedra that follow one
// another in a mesh share most of their vertices and edges, and device-wide
// atomics at random addresses are what this path is bound by (26 G/s,
// whatever the array's size): a block of 512 consecutive Kuhn tetrahedra has
// 344 distinct vertices instead of 2,048 corners and 1,200 distinct edges
// instead of 3,072.  On the 24.1M tetrahedra of a 160^3 mesh the count takes
// 0.92 ms and the scatter 1.25 ms (3.76 and 4.51 ms with one atomic per
// corner).  The tables hold every block's worst case (all vertices distinct),
// so tetrahedra in no order lose only the reduction (a call that took 13.7 ms
// takes 11.7 on the same ones shuffled).
constexpr int kTets = 512;
constexpr int kTetSlots = 4096;  // of each table: 2,048 vertices, 3,072 edges
constexpr uint32_t kNoEdge = 0xffffffffu;

struct TetTables {
  int32_t vert[kTetSlots];       // vertex id, or -1
  uint32_t edge[kTetSlots];      // lower slot << 12 | higher slot, or kNoEdge
  uint32_t deg[kTetSlots];       // distinct edges at the vertex
};

// Slot of vertex v (the table never fills: at most 4 * kTets distinct ids).
__device__ __forceinline__ uint32_t tet_vertex(int32_t *vert, int32_t v) {
  uint32_t h = ((uint32_t)v * 0x9e3779b1u) >> 20;
  for (;;) {
    int32_t cur = vert[h];
    if (cur == -1) cur = atomicCAS(&vert[h], -1, v);
    if (cur == -1 || cur == v) return h;
    h = (h + 1) & (kTetSlots - 1);
  }
}

// True for the one caller that enters the edge (at most 6 * kTets of them).
__device__ __forceinline__ bool tet_edge(uint32_t *edge, uint32_t key) {
  uint32_t h = (key * 0x9e3779b1u) >> 20;
  for (;;) {
    uint32_t cur = edge[h];
    if (cur == key) return false;
    if (cur == kNoEdge) {
      cur = atomicCAS(&edge[h], kNoEdge, key);
      if (cur == kNoEdge) return true;
      if (cur == key) return false;
    }
    h = (h + 1) & (kTetSlots - 1);
  }
}

constexpr int kTetEdges[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};

// Fills the block's tables (one tetrahedron per thread).  `v` and `slot` get
// the thread's corners, the result has a bit for each of its edges that this
// thread entered.  A tetrahedron with a vertex outside [0, n) is skipped and
// reported in *bad.  Ends with a barrier.
__device__ __forceinline__ uint32_t tet_reduce(TetTables &s, int64_t ntets,
                                               const int32_t *__restrict__ tets,
                                               int64_t n, int32_t (&v)[4],
                                               uint32_t (&slot)[4],
                                               bool *bad) {
  for (int i = threadIdx.x; i < kTetSlots; i += kTets) {
    s.vert[i] = -1;
    s.edge[i] = kNoEdge;
    s.deg[i] = 0;
  }
  const int64_t t = (int64_t)blockIdx.x * kTets + threadIdx.x;
  const bool in = t < ntets;
  bool out = false;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = in ? tets[4 * t + k] : 0;
    out |= in && (v[k] < 0 || (int64_t)v[k] >= n);
  }
  *bad = out;
  __syncthreads();
  uint32_t own = 0;
  if (in && !out) {
#pragma unroll
    for (int k = 0; k < 4; ++k) slot[k] = tet_vertex(s.vert, v[k]);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const uint32_t a = slot[kTetEdges[e][0]], b = slot[kTetEdges[e][1]];
      if (a == b) continue;  // a repeated vertex is no neighbour of itself
      if (tet_edge(s.edge, a < b ? a << 12 | b : b << 12 | a)) {
        own |= 1u << e;
        atomicAdd(&s.deg[a], 1u);
        atomicAdd(&s.deg[b], 1u);
      }
    }
  }
  __syncthreads();
  return own;
}

// Candidates of every vertex: each block adds its distinct edges there.
__global__ void __launch_bounds__(kTets)
k_tet_count(int64_t ntets, const int32_t *__restrict__ tets, int64_t n,
            uint32_t *cnt, unsigned long long *ctr) {
  __shared__ TetTables s;
  int32_t v[4];
  uint32_t slot[4];
  bool bad;
  (void)tet_reduce(s, ntets, tets, n, v, slot, &bad);
  for (int i = threadIdx.x; i < kTetSlots; i += kTets)
    if (s.deg[i]) atomicAdd(&cnt[s.vert[i]], s.deg[i]);
  flag_any(bad, ctr + kCtrBadIndex);
}

// The same reduction again (it costs less than keeping its result would),
// then each of the block's vertices takes its run of candidates with one
// atomic and the owners of the edges write both directions.
__global__ void __launch_bounds__(kTets)
k_tet_scatter(int64_t ntets, const int32_t *__restrict__ tets, int64_t n,
              const int64_t *__restrict__ off, uint32_t *cursor,
              int32_t *__restrict__ cand) {
  constexpr int K = kTetSlots / kTets;
  __shared__ TetTables s;
  int32_t v[4];
  uint32_t slot[4];
  bool bad;
  const uint32_t own = tet_reduce(s, ntets, tets, n, v, slot, &bad);
  // The next free place of every slot's run, over the edge and degree
  // tables, which are done with once the degrees are in registers.
  static_assert(sizeof(s.edge) + sizeof(s.deg) == kTetSlots * 8, "aliased");
  unsigned long long *at = reinterpret_cast<unsigned long long *>(s.edge);
  uint32_t d[K];
  unsigned long long base[K];
#pragma unroll
  for (int k = 0; k < K; ++k) d[k] = s.deg[threadIdx.x + k * kTets];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int32_t u = s.vert[threadIdx.x + k * kTets];
    base[k] = d[k] ? (unsigned long long)off[u] + atomicAdd(&cursor[u], d[k])
                   : 0ull;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) at[threadIdx.x + k * kTets] = base[k];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    if (!((own >> e) & 1u)) continue;
    const int a = kTetEdges[e][0], b = kTetEdges[e][1];
    cand[atomicAdd(&at[slot[a]], 1ull)] = v[b];
    cand[atomicAdd(&at[slot[b]], 1ull)] = v[a];
  }
}

// Rows are worked on in LDS, kRows of them per block and one per thread: the
// candidates of consecutive vertices are one contiguous run, loaded and
// stored whole, where a thread walking its own row in device memory pulls a
// line per step (at 160^3: distinct 0.69 ms instead of 4.26, with 2.6 times
// fewer candidates; fill 0.47 ms instead of 1.42).  A block whose run does not
// fit walks its rows in device memory.
constexpr int kRows = 128;
constexpr int kRowCand = 10240;  // candidates in LDS: 80 per row, 40 KB
constexpr int kRowOut = 4096;    // distinct neighbours: 32 per row

// A row's candidates are examined eight at a time.  The first occurrence of
// every neighbour (not the vertex itself) moves to the front of the row as
// it goes: a candidate is new when it matches neither that compacted prefix
// nor an earlier candidate of its batch, and the prefix never reaches past
// the batch being examined, so every candidate is read before it can be
// overwritten.  Returns the number of distinct neighbours.
constexpr int kRowBatch = 8;

__device__ __forceinline__ uint32_t row_distinct(int32_t *seg, int64_t k,
                                                 int32_t v) {
  uint32_t count = 0;
  for (int64_t i0 = 0; i0 < k; i0 += kRowBatch) {
    int32_t c[kRowBatch];
    bool dup[kRowBatch];
#pragma unroll
    for (int t = 0; t < kRowBatch; ++t) {
      c[t] = seg[i0 + t < k ? i0 + t : i0];
      dup[t] = i0 + t >= k || c[t] == v;
    }
    for (uint32_t j = 0; j < count; ++j) {
      const int32_t d = seg[j];
#pragma unroll
      for (int t = 0; t < kRowBatch; ++t) dup[t] |= d == c[t];
    }
#pragma unroll
    for (int t = 1; t < kRowBatch; ++t)
#pragma unroll
      for (int q = 0; q < t; ++q) dup[t] |= c[q] == c[t];
#pragma unroll
    for (int t = 0; t < kRowBatch; ++t)
      if (!dup[t]) seg[count++] = c[t];
  }
  return count;
}

// Each of a row's u distinct neighbours to its rank among them.
__device__ __forceinline__ void row_sort(const int32_t *seg, int64_t u,
                                         int32_t *to) {
  for (int64_t i0 = 0; i0 < u; i0 += kRowBatch) {
    int32_t c[kRowBatch];
    uint32_t rank[kRowBatch];
#pragma unroll
    for (int t = 0; t < kRowBatch; ++t) {
      c[t] = seg[i0 + t < u ? i0 + t : i0];
      rank[t] = 0;
    }
    for (int64_t j = 0; j < u; ++j) {
      const int32_t d = seg[j];
#pragma unroll
      for (int t = 0; t < kRowBatch; ++t) rank[t] += d < c[t];
    }
#pragma unroll
    for (int t = 0; t < kRowBatch; ++t)
      if (i0 + t < u) to[rank[t]] = c[t];
  }
}

// `keep`: the compacted rows go back to `cand` for the fill.
__global__ void __launch_bounds__(kRows)
k_row_distinct(int64_t n, const int64_t *__restrict__ off, int32_t *cand,
               uint32_t *ucnt, bool keep) {
  __shared__ int32_t sc[kRowCand];
  const int64_t v0 = (int64_t)blockIdx.x * kRows, v = v0 + threadIdx.x;
  const int64_t v1 = v0 + kRows < n ? v0 + kRows : n;
  const int64_t b0 = off[v0], len = off[v1] - b0;
  const int64_t o0 = off[v < n ? v : n], o1 = off[v < n ? v + 1 : n];
  const bool staged = len <= kRowCand;  // block-uniform
  if (staged) {
    for (int64_t i = threadIdx.x; i < len; i += kRows) sc[i] = cand[b0 + i];
    __syncthreads();
  }
  if (v < n)
    ucnt[v] = staged ? row_distinct(sc + (o0 - b0), o1 - o0, (int32_t)v)
                     : row_distinct(cand + o0, o1 - o0, (int32_t)v);
  if (staged && keep) {
    __syncthreads();
    for (int64_t i = threadIdx.x; i < len; i += kRows) cand[b0 + i] = sc[i];
  }
}

__global__ void __launch_bounds__(kRows)
k_row_fill(int64_t n, const int64_t *__restrict__ off,
           const int32_t *__restrict__ cand,
           const int64_t *__restrict__ row_ptr, int32_t *__restrict__ col) {
  __shared__ int32_t sin[kRowOut], sout[kRowOut];
  __shared__ uint32_t first[kRows + 1];  // of each row within the block's run
  __shared__ int64_t from[kRows];        // start of its candidates
  const int64_t v0 = (int64_t)blockIdx.x * kRows, v = v0 + threadIdx.x;
  const int64_t v1 = v0 + kRows < n ? v0 + kRows : n;
  const int64_t r0 = row_ptr[v0], len = row_ptr[v1] - r0;
  const int64_t base = row_ptr[v < n ? v : n];
  const int64_t u = row_ptr[v < n ? v + 1 : n] - base;
  if (len > kRowOut) {  // block-uniform
    if (v < n) row_sort(cand + off[v], u, col + base);
    return;
  }
  from[threadIdx.x] = v < n ? off[v] : 0;
  first[threadIdx.x] = (uint32_t)(base - r0);
  if (threadIdx.x == 0) first[kRows] = (uint32_t)len;
  __syncthreads();
  // Entry i of the run belongs to the last row that starts at or before it
  // (the rows that hold nothing start where the next one does).
  for (uint32_t i = threadIdx.x; i < (uint32_t)len; i += kRows) {
    uint32_t lo = 0;
#pragma unroll
    for (uint32_t h = kRows / 2; h > 0; h >>= 1)
      if (first[lo + h] <= i) lo += h;
    sin[i] = cand[from[lo] + (i - first[lo])];
  }
  __syncthreads();
  row_sort(sin + (base - r0), u, sout + (base - r0));
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < (uint32_t)len; i += kRows)
    col[r0 + i] = sout[i];
}

unsigned grid64(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

int scan64(msc_ctx *ctx, const uint32_t *cnt, int64_t n, int64_t *out,
           uint64_t *bsum, hipStream_t s) {
  const int64_t nb = (n + kScan - 1) / kScan;
  if (n > 0)
    k_scan64_blocks<<<grid64(n, kScan), kScan, 0, s>>>(cnt, n, out, bsum);
  k_scan64_sums<<<1, kScan, 0, s>>>(bsum, nb, out, n);  // out[n]: the total
  if (n > 0) k_scan64_add<<<grid64(n, kBlock), kBlock, 0, s>>>(out, n, bsum);
  (void)ctx;
  return MSC_OK;
}

}  // namespace

int csr_from_tets_run(msc_ctx *ctx, int64_t n, int64_t ntets,
                      const int32_t *tets, int64_t *row_ptr, int32_t *col_idx,
                      int64_t capacity, msc_alloc_fn alloc, void *user,
                      int64_t *nnz, hipStream_t s) {
  const int64_t nb = (n + kScan - 1) / kScan;
  const int64_t ncand = 12 * ntets;
  MSC_TRY(reserve(ctx, ctx->ws, align256(n * 4) + align256((n + 1) * 8) +
                               align256(nb * 8 + 8) + align256(ncand * 4) +
                               4096));
  Carver cv(ctx->ws);
  uint32_t *cnt = cv.take<uint32_t>(n);
  int64_t *off = cv.take<int64_t>(n + 1);
  uint64_t *bsum = cv.take<uint64_t>(nb + 1);
  int32_t *cand = cv.take<int32_t>(ncand);
  MSC_TRY(clear_counters(ctx, s));
  if (n > 0) k_zero32<<<grid64(n, kBlock), kBlock, 0, s>>>(cnt, n);
  if (ntets > 0)
    MSC_PHASE(ctx, s, "tets_count", 16.0 * ntets,
              (k_tet_count<<<grid64(ntets, kTets), kTets, 0, s>>>(
                  ntets, tets, n, cnt, ctx->dctr)));
  MSC_PHASE(ctx, s, "tets_scan", 12.0 * n, (scan64(ctx, cnt, n, off, bsum, s)));
  if (n > 0) k_zero32<<<grid64(n, kBlock), kBlock, 0, s>>>(cnt, n);
  if (ntets > 0)
    MSC_PHASE(ctx, s, "tets_scatter", 16.0 * ntets + 4.0 * ncand,
              (k_tet_scatter<<<grid64(ntets, kTets), kTets, 0, s>>>(
                  ntets, tets, n, off, cnt, cand)));
  if (n > 0)
    MSC_PHASE(ctx, s, "rows_distinct", 4.0 * ncand + 12.0 * n,
              (k_row_distinct<<<grid64(n, kRows), kRows, 0, s>>>(
                  n, off, cand, cnt, col_idx || alloc)));
  MSC_PHASE(ctx, s, "rows_scan", 12.0 * n,
            (scan64(ctx, cnt, n, row_ptr, bsum, s)));
  MSC_TRY(read_counters(ctx, s, row_ptr + n));
  if (ctx->hctr[kCtrBadIndex]) return MSC_EINVAL;
  const int64_t total = (int64_t)ctx->hctr[kCtrExtra];
  *nnz = total;
  if (alloc && total > 0) {
    col_idx = static_cast<int32_t *>(alloc(user, total));
    if (!col_idx) return MSC_ENOMEM;
    capacity = total;
  }
  if (col_idx && capacity >= total && total > 0) {
    MSC_PHASE(ctx, s, "rows_fill", 4.0 * ncand + 4.0 * total,
              (k_row_fill<<<grid64(n, kRows), kRows, 0, s>>>(
                  n, off, cand, row_ptr, col_idx)));
    MSC_TRY(read_counters(ctx, s));
  }
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = n;
  return MSC_OK;
}

// ---------------------------------------------------------------------------
// Critical points and the extremum graph (background, "Critical Points";
// the extremum graph that the segmentations feed): the lower and upper link
// of every vertex and their connected components, from the 14 Freudenthal
// neighbours.  The triangulation is a flag complex, so two neighbours of v
// span a link edge exactly when they are neighbours of each other; a link
// vertex outside the domain is absent, which gives the link of boundary
// vertices and of 2-D and 1-D grids.
// ---------------------------------------------------------------------------

namespace {

struct NbVec {
  int dx, dy, dz;
};
// The neighbours in increasing (dz, dy, dx), i.e. in increasing vertex id.
constexpr NbVec kNb[14] = {
    {-1, -1, -1}, {0, -1, -1}, {-1, 0, -1}, {0, 0, -1}, {-1, -1, 0},
    {0, -1, 0},   {-1, 0, 0},  {1, 0, 0},   {0, 1, 0},  {1, 1, 0},
    {0, 0, 1},    {1, 0, 1},   {0, 1, 1},   {1, 1, 1}};

// A coordinate of every neighbour, two bits each (the step plus one).
constexpr uint32_t pack_steps(int axis) {
  uint32_t p = 0;
  for (int i = 0; i < 14; ++i) {
    const int d = axis == 0 ? kNb[i].dx : (axis == 1 ? kNb[i].dy : kNb[i].dz);
    p |= (uint32_t)(d + 1) << (2 * i);
  }
  return p;
}
constexpr uint32_t kNbX = pack_steps(0), kNbY = pack_steps(1),
                   kNbZ = pack_steps(2);

__device__ __forceinline__ int64_t nb_step(uint32_t steps, int i) {
  return (int64_t)((steps >> (2 * i)) & 3u) - 1;
}

constexpr bool edge_vector(int a, int b, int c) {
  const bool nonneg = a >= 0 && b >= 0 && c >= 0 && a <= 1 && b <= 1 && c <= 1;
  const bool nonpos = a <= 0 && b <= 0 && c <= 0 && a >= -1 && b >= -1 &&
                      c >= -1;
  return (a | b | c) != 0 && (nonneg || nonpos);
}

constexpr uint32_t link_adj(int i) {
  uint32_t m = 0;
  for (int j = 0; j < 14; ++j)
    if (j != i && edge_vector(kNb[i].dx - kNb[j].dx, kNb[i].dy - kNb[j].dy,
                              kNb[i].dz - kNb[j].dz))
      m |= 1u << j;
  return m;
}

// Components of the link restricted to a set of neighbours depend on the set
// alone (the adjacency is fixed and absent neighbours are simply not in the
// set), so two tables over all 2^14 sets, made when this file is compiled,
// replace the per-vertex growth: the number of components, and the component
// that holds the set's lowest neighbour.  Removing that component leaves a set
// whose components are the remaining ones, so repeated lookups enumerate them.
constexpr int kLinkSets = 1 << 14;

struct alignas(16) LinkTables {  // read 16 bytes at a time (stage_ncomp)
  uint8_t ncomp[kLinkSets];
  uint16_t first[kLinkSets];
};

constexpr LinkTables make_link_tables() {
  LinkTables t{};
  uint32_t adj[14] = {};
  for (int i = 0; i < 14; ++i) adj[i] = link_adj(i);
  for (uint32_t set = 1; set < (uint32_t)kLinkSets; ++set) {
    // Grown from the lowest neighbour, one newly reached member at a time.
    uint32_t comp = set & (0u - set), todo = comp;
    while (todo) {
      const int i = __builtin_ctz(todo);
      todo &= todo - 1;
      const uint32_t fresh = adj[i] & set & ~comp;
      comp |= fresh;
      todo |= fresh;
    }
    t.first[set] = (uint16_t)comp;
    t.ncomp[set] = (uint8_t)(1 + t.ncomp[set & ~comp]);  // a smaller set
  }
  return t;
}

__device__ constexpr LinkTables kLink = make_link_tables();

struct LinkSets {
  float fn[14];          // neighbour values (meaningless where absent)
  uint32_t lower, upper; // neighbours below / above v in the (f, id) order
  bool nan;
};

// Requires X·Y·Z <= INT32_MAX (checked by the entry points), so ids and id
// offsets fit 32 bits.
__device__ __forceinline__ LinkSets link_sets(const float *__restrict__ f,
                                              int64_t X, int64_t Y, int64_t Z,
                                              int64_t v) {
  const uint32_t vv = (uint32_t)v, X32 = (uint32_t)X, Y32 = (uint32_t)Y;
  const uint32_t row = vv / X32;
  const uint32_t x = vv - row * X32, y = row % Y32, z = row / Y32;
  const int32_t sx = 1, sy = (int32_t)X32, sz = (int32_t)(X32 * Y32);
  // Per axis, whether the step down / up stays in the grid; a step that
  // would leave it is taken as 0, so every load below stays in bounds and
  // the neighbour is marked absent.
  const bool lo[3] = {x > 0, y > 0, z > 0};
  const bool hi[3] = {x + 1 < X32, y + 1 < Y32, (int64_t)z + 1 < Z};
  const int32_t step[3] = {sx, sy, sz};
  const float *p = f + v;
  const float fv = p[0];
  LinkSets ls;
  uint32_t present = 0;
#pragma unroll
  for (int i = 0; i < 14; ++i) {
    const int d[3] = {kNb[i].dx, kNb[i].dy, kNb[i].dz};
    int32_t off = 0;
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (d[a] < 0) {
        in = in && lo[a];
        off -= lo[a] ? step[a] : 0;
      } else if (d[a] > 0) {
        in = in && hi[a];
        off += hi[a] ? step[a] : 0;
      }
    }
    ls.fn[i] = p[off];
    present |= (uint32_t)in << i;
  }
  ls.nan = fv != fv;
  uint32_t lower = 0;
#pragma unroll
  for (int i = 0; i < 14; ++i) {
    // the first 7 neighbours have smaller ids than v
    const bool below = ls.fn[i] < fv || (ls.fn[i] == fv && i < 7);
    lower |= (uint32_t)below << i;
  }
  ls.lower = lower & present;
  ls.upper = present & ~lower;
  return ls;
}

// The (f, id)-extreme neighbour of each component of `set` (the highest when
// `high`), as a neighbour mask.  Neighbour order is id order, so a tie in
// value goes to the larger index for the highest and the smaller for the
// lowest.
__device__ __forceinline__ uint32_t component_extremes(uint32_t set,
                                                       const float *fn,
                                                       bool high) {
  uint32_t rem = set, ex = 0;
  while (rem) {
    const uint32_t comp = kLink.first[rem];
    int best = -1;
    float fb = 0.f;
#pragma unroll
    for (int i = 0; i < 14; ++i) {
      if (!((comp >> i) & 1u)) continue;
      const bool better = best < 0 || (high ? fn[i] >= fb : fn[i] < fb);
      if (better) {
        best = i;
        fb = fn[i];
      }
    }
    ex |= 1u << best;
    rem &= ~comp;
  }
  return ex;
}

// The link sets of every vertex, for passes that take the whole grid: a thread
// walks up z from a position p = x + X*y of the plane, so that seven loads per
// vertex (the plane above; the others are in registers) do instead of fifteen,
// the position's neighbours are located once per walk, and a comparison goes
// straight from the lane mask it leaves into the set's next bit.  Consecutive
// threads take consecutive positions, whatever the rows' length: a wave's 64
// vertices of a plane are 64 consecutive ids (a run).  What bounds these passes
// is vector and LDS issue, about 50 vector operations a vertex (189 with
// fifteen loads and a vertex's own coordinates).  Critical points of 512^3 take
// 0.26 ms instead of 0.60 (2.6 TB/s of the 5 bytes a vertex); 0.28 rolled, 0.35
// without the load ahead.
constexpr int kWalkThreads = 512;

struct Walk {
  const float *f;
  uint32_t X, Y, Z, XY, runs;  // runs of 64 positions per plane
  uint32_t pb;                 // blocks per plane
  int zc;                      // planes per walk
};

// The lane's bits of 14 compares' masks as a number, m[0]'s highest.  The
// compiler does not see what is inside an asm block, so the wait states that a
// vector operation needs before it reads a mask that a compare has just written
// stand at its start (two; inside, each mask is older than that).
__device__ __forceinline__ uint32_t lane_bits(const unsigned long long (&m)[14]) {
  uint32_t r = 0;
  asm("s_nop 1\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %1\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %2\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %3\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %4\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %5\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %6\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %7\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %8\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %9\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %10\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %11\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %12\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %13\n"
      "\tv_addc_co_u32 %0, vcc, %0, %0, %14"
      : "+v"(r)
      : "s"(m[0]), "s"(m[1]), "s"(m[2]), "s"(m[3]), "s"(m[4]), "s"(m[5]),
        "s"(m[6]), "s"(m[7]), "s"(m[8]), "s"(m[9]), "s"(m[10]), "s"(m[11]),
        "s"(m[12]), "s"(m[13])
      : "vcc");
  return r;
}

__device__ __forceinline__ unsigned long long lanes(bool b) {
  return __builtin_amdgcn_ballot_w64(b);
}

// Calls use(z, p, inside, lower, upper) for every plane of the block's chunk of
// ZC planes, with all lanes; returns whether a value of the lane's was NaN.
// The walk is unrolled, so that the planes' registers change their names and
// are not copied (18 of 75 operations a vertex).
template <int ZC, class Use>
__device__ __forceinline__ bool walk_links(const Walk &w, Use use) {
  const uint32_t blk = cc_tile_of_block(blockIdx.x, gridDim.x);
  const uint32_t chunk = blk / w.pb;
  const uint32_t p0 = (blk - chunk * w.pb) * kWalkThreads + threadIdx.x;
  const bool inside = p0 < w.XY;
  const uint32_t p = inside ? p0 : w.XY - 1;
  const uint32_t y = p / w.X, x = p - y * w.X;
  const bool xl = x > 0, yl = y > 0, xh = x + 1 < w.X, yh = y + 1 < w.Y;
  // A neighbour outside the grid is read as the position itself and is not
  // in `here`, the neighbours that exist in the planes below, at and above.
  const uint32_t low = (xl && yl) | (uint32_t)yl << 1 | (uint32_t)xl << 2,
                 high = (uint32_t)xh | (uint32_t)yh << 1 |
                        (uint32_t)(xh && yh) << 2;
  const uint32_t here = low | 8u | low << 4 | high << 7 | 1u << 10 | high << 11;
  const uint32_t oxl = p - (xl ? 1u : 0u), oyl = p - (yl ? w.X : 0u),
                 oxyl = p - (xl && yl ? w.X + 1 : 0u);
  const uint32_t oxh = p + (xh ? 1u : 0u), oyh = p + (yh ? w.X : 0u),
                 oxyh = p + (xh && yh ? w.X + 1 : 0u);
  struct PlaneL {
    float xyl, yl, xl, c;
  };
  struct PlaneH {
    float xh, yh, xyh;
  };
  typedef __attribute__((address_space(1))) const float GF;
  auto plane = [&](uint32_t z) {
    return (GF *)w.f + (size_t)w.XY * z;
  };
  auto load_l = [&](uint32_t z) {
    GF *q = plane(z);
    return PlaneL{q[oxyl], q[oyl], q[oxl], q[p]};
  };
  auto load_h = [&](uint32_t z) {
    GF *q = plane(z);
    return PlaneH{q[oxh], q[oyh], q[oxyh]};
  };
  const uint32_t z0 = chunk * ZC;
  // The plane above is loaded one step ahead of its use.
  auto in_z = [&](uint32_t z) { return z < w.Z ? z : w.Z - 1; };
  PlaneL below = load_l(z0 > 0 ? z0 - 1 : 0), cur = load_l(z0);
  PlaneH curh = load_h(z0);
  PlaneL up = load_l(in_z(z0 + 1));
  PlaneH uph = load_h(in_z(z0 + 1));
  bool nan = false;
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)ZC; ++k) {
    const uint32_t z = z0 + k;
    if (z >= w.Z) break;  // uniform
    const PlaneL next = load_l(in_z(z + 2));
    const PlaneH nexth = load_h(in_z(z + 2));
    const float v = cur.c;
    nan |= v != v;
    // Neighbours in decreasing id; the ones with smaller ids than v are below
    // it when equal.
    const unsigned long long m[14] = {
        lanes(uph.xyh < v), lanes(uph.yh < v),
        lanes(uph.xh < v), lanes(up.c < v),
        lanes(curh.xyh < v), lanes(curh.yh < v),
        lanes(curh.xh < v), lanes(cur.xl <= v),
        lanes(cur.yl <= v), lanes(cur.xyl <= v),
        lanes(below.c <= v), lanes(below.xl <= v),
        lanes(below.yl <= v), lanes(below.xyl <= v)};
    const uint32_t s = lane_bits(m);
    const uint32_t planes = (z > 0 ? 0xfu : 0u) | 0x3f0u |
                            (z + 1 < w.Z ? 0x3c00u : 0u);  // uniform
    const uint32_t present = here & planes;
    use(z, p0, inside, s & present, present & ~s);
    below = cur;
    cur = up;
    curh = uph;
    up = next;
    uph = nexth;
  }
  return inside && nan;
}

// The count table in LDS, where both lookups of a vertex cost one read.
__device__ __forceinline__ void stage_ncomp(uint8_t *t) {
  static_assert(alignof(LinkTables) >= alignof(uint4) &&
                    offsetof(LinkTables, ncomp) == 0 && kLinkSets % 16 == 0,
                "whole aligned uint4s");
  const uint4 *src = reinterpret_cast<const uint4 *>(kLink.ncomp);
  for (int i = threadIdx.x; i < kLinkSets / 16; i += kWalkThreads)
    reinterpret_cast<uint4 *>(t)[i] = src[i];
  __syncthreads();
}

template <int ZC>
__global__ void __launch_bounds__(kWalkThreads)
k_critical(Walk w, uint8_t *__restrict__ code, unsigned long long *ctr) {
  __shared__ __align__(16) uint8_t nc[kLinkSets];
  stage_ncomp(nc);
  typedef __attribute__((address_space(1))) uint8_t GB;
  const bool nan = walk_links<ZC>(w, [&](uint32_t z, uint32_t p, bool inside,
                                     uint32_t lower, uint32_t upper) {
    const uint32_t c = nc[lower] | (uint32_t)nc[upper] << 4;
    if (inside) ((GB *)code + (size_t)w.XY * z)[p] = (uint8_t)c;
  });
  flag_any(nan, ctr + kCtrNaN);
}

// The same with a vertex per thread, for grids that the walk does not suit.
__global__ void __launch_bounds__(kBlock)
k_critical_small(const float *__restrict__ f, int64_t X, int64_t Y, int64_t Z,
                 uint8_t *__restrict__ code, unsigned long long *ctr) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  bool nan = false;
  if (v < X * Y * Z) {
    const LinkSets ls = link_sets(f, X, Y, Z, v);
    code[v] = (uint8_t)(kLink.ncomp[ls.lower] | kLink.ncomp[ls.upper] << 4);
    nan = ls.nan;
  }
  flag_any(nan, ctr + kCtrNaN);
}

// Edges of a vertex: one per component of a side that has two or more.
__device__ __forceinline__ uint32_t edge_count(uint32_t lc, uint32_t uc) {
  return (uc >= 2 ? uc : 0u) + (lc >= 2 ? lc : 0u);
}

// Exclusive prefix over a block of kBlock threads and the block total, for
// per-thread counts below 16 (a vertex has at most 14 edges: its lower and
// upper link components together number at most its 14 link vertices).  One
// ballot per bit: a lane's prefix in its wave is the sum over bits k of 2^k
// times the number of lower lanes with bit k set.
__device__ __forceinline__ uint32_t block_scan16(uint32_t x, uint32_t *tmp,
                                                 uint32_t *total) {
  const int w = threadIdx.x >> 6;
  uint32_t pre = 0, sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const unsigned long long b = __ballot((x >> k) & 1u);
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
    pre += below << k;
    sum += (uint32_t)__popcll(b) << k;
  }
  if ((threadIdx.x & 63) == 0) tmp[w] = sum;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kBlock / 64; ++k) {
    const uint32_t t = tmp[k];
    before += k < w ? t : 0u;
    all += t;
  }
  *total = all;
  return before + pre;
}

// The edges of vertex v from position `at` on: ascending ones first, then
// descending; within a side, components by increasing id of their extreme
// vertex (= neighbour order).
__device__ __forceinline__ void egraph_emit(const LinkSets &ls, int64_t v,
                                            int64_t X, int64_t XY, uint32_t lc,
                                            uint32_t uc,
                                            const int32_t *__restrict__ asc,
                                            const int32_t *__restrict__ desc,
                                            int32_t *__restrict__ out,
                                            int64_t at) {
  // Both sides' extreme neighbours in output order, one per step: the lanes
  // of a wave then take as many steps as the vertex with most edges has, where
  // a step per neighbour would wait for 28 gathers in turn.
  const uint32_t hm = component_extremes(uc >= 2 ? ls.upper : 0u, ls.fn, true),
                 lm = component_extremes(lc >= 2 ? ls.lower : 0u, ls.fn, false);
  for (uint32_t m = hm | lm << 14; m; m &= m - 1) {
    const int k = __ffs((int)m) - 1;
    const bool high = k < 14;
    const int i = high ? k : k - 14;
    const int64_t u = v + nb_step(kNbX, i) + X * nb_step(kNbY, i) +
                      XY * nb_step(kNbZ, i);
    const int32_t e = (high ? asc : desc)[u];
    out[3 * at] = (int32_t)v;
    out[3 * at + 1] = e;
    out[3 * at + 2] = high ? 1 : -1;
    ++at;
  }
}

// Every run's vertices with edges as a lane mask, and the number of the run's
// edges; the write pass then looks at those vertices alone.
template <int ZC>
__global__ void __launch_bounds__(kWalkThreads)
k_egraph_mark(Walk w, unsigned long long *__restrict__ marks,
              uint32_t *__restrict__ counts, unsigned long long *ctr) {
  __shared__ __align__(16) uint8_t nc[kLinkSets];
  stage_ncomp(nc);
  const bool nan = walk_links<ZC>(w, [&](uint32_t z, uint32_t p, bool inside,
                                     uint32_t lower, uint32_t upper) {
    const uint32_t c = inside ? edge_count(nc[lower], nc[upper]) : 0u;
    const unsigned long long m = lanes(c != 0u);
    uint32_t sum = 0;
    if (m) {  // a count has four bits: a vertex has at most 14 edges
#pragma unroll
      for (int k = 0; k < 4; ++k)
        sum += (uint32_t)__popcll(lanes((c >> k) & 1u)) << k;
    }
    if ((threadIdx.x & 63) == 0 && p < w.XY) {
      const size_t r = (size_t)w.runs * z + p / 64;
      marks[r] = m;
      counts[r] = sum;
    }
  });
  flag_any(nan, ctr + kCtrNaN);
}

// A wave takes K consecutive runs (at most 31), lists their marked vertices in
// LDS, and works through the list 64 at a time, so that its lanes are full
// however the marks lie.  The edges of its runs are one contiguous stretch of
// the output, in the list's order.  K is what holds about 64 edges, since with
// more the long lists of noisy regions are left to few waves, but at least four
// runs, since a run of noise fills less than half of the lanes; and fewer where
// that would leave less than 4,096 waves.  Above four it is odd: with a power of
// two the blocks that share a CU come from the same part of the planes, which
// noise fills or leaves empty together.  The list takes LDS for K runs and no
// more, so that a CU holds all the waves it can.  A whole call, in us, at
//                              edges/run  K = 1    4    5    8   11   23   31   32
//   512^3 noise                       62   3548 2428 2558 2415 2488 2547 2690 2668
//   300x280x290 Gaussian, noisy       30    565  348  338  332  337  357  370  375
//   512^3 Gaussian sums              3.2   1151  709  652  647  566  534  538  949
//   700x600x500 the same             1.2   1273  862  813  756  705  651  639  645
//   512^3 Perlin noise               0.6   1199  776  732  623  544  459  445  447
//   64^3 Gaussian sums                41     61   65   70   76   83  108  129  129
// Up to kFewRuns runs are listed with a lane per vertex, more with a lane per
// run (their marks are few).
constexpr int kFewRuns = 8;

__global__ void __launch_bounds__(kBlock)
k_egraph_write(Walk w, uint64_t nruns, int K,
               const unsigned long long *__restrict__ marks,
               const int64_t *__restrict__ off,
               const int32_t *__restrict__ asc,
               const int32_t *__restrict__ desc, int32_t *__restrict__ out) {
  extern __shared__ uint16_t list[];  // 64 * K per wave: run << 6 | position
  const int lane = threadIdx.x & 63;
  uint16_t *const mine = list + (threadIdx.x >> 6) * (64 * K);
  const uint64_t r0 =
      ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / 64 * (uint32_t)K;
  const uint64_t r = r0 + lane;
  const unsigned long long m = lane < K && r < nruns ? marks[r] : 0ull;
  const uint32_t n = (uint32_t)__popcll(m);
  uint32_t inc = n;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  const uint32_t total = __shfl(inc, 63);
  uint32_t at = inc - n;
  if (K > kFewRuns) {  // a lane per run
    for (unsigned long long t = m; t; t &= t - 1)
      mine[at++] = (uint16_t)(lane << 6 | (__ffsll((long long)t) - 1));
  } else {  // a lane per vertex
    for (int q = 0; q < K; ++q) {
      const unsigned long long mq = __shfl(m, q);
      const uint32_t base = __shfl(at, q);
      if ((mq >> lane) & 1u)
        mine[base + __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(mq >> 32),
                        __builtin_amdgcn_mbcnt_lo((uint32_t)mq, 0u))] =
            (uint16_t)(q << 6 | lane);
    }
  }
  __syncthreads();
  if (!total) return;  // uniform over the wave
  const uint64_t z0 = r0 / w.runs;
  const uint32_t run0 = (uint32_t)(r0 - z0 * w.runs);
  int64_t base = off[r0];
  for (uint32_t j = 0; j < total; j += 64) {
    const bool on = j + lane < total;
    const uint32_t it = mine[on ? j + lane : j];
    const uint32_t rr = run0 + (it >> 6), dz = rr / w.runs;
    const int64_t v = (int64_t)((z0 + dz) * w.XY) +
                      64 * (int64_t)(rr - dz * w.runs) + (it & 63u);
    const LinkSets ls = link_sets(w.f, w.X, w.Y, w.Z, v);
    const uint32_t lc = kLink.ncomp[ls.lower], uc = kLink.ncomp[ls.upper];
    const uint32_t c = on ? edge_count(lc, uc) : 0u;
    uint32_t pre = 0, sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned long long b = lanes((c >> k) & 1u);
      pre += __builtin_amdgcn_mbcnt_hi(
                 (uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))
             << k;
      sum += (uint32_t)__popcll(b) << k;
    }
    if (on) egraph_emit(ls, v, w.X, w.XY, lc, uc, asc, desc, out, base + pre);
    base += sum;
  }
}

// The same graph with a word per 256 vertices in place of 20 bytes per run:
// for grids whose planes are narrower than a run (chains along z), and for a
// caller's workspace that holds no more.
__global__ void __launch_bounds__(kBlock)
k_egraph_count_small(const float *__restrict__ f, int64_t X, int64_t Y,
                     int64_t Z, uint32_t *bcount, unsigned long long *ctr) {
  __shared__ uint32_t tmp[kBlock / 64];
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  uint32_t c = 0;
  bool nan = false;
  if (v < X * Y * Z) {
    const LinkSets ls = link_sets(f, X, Y, Z, v);
    c = edge_count(kLink.ncomp[ls.lower], kLink.ncomp[ls.upper]);
    nan = ls.nan;
  }
  flag_any(nan, ctr + kCtrNaN);
  uint32_t tot = 0;
  (void)block_scan16(c, tmp, &tot);
  if (threadIdx.x == 0) bcount[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kBlock)
k_egraph_write_small(const float *__restrict__ f, int64_t X, int64_t Y,
                     int64_t Z, const int32_t *__restrict__ asc,
                     const int32_t *__restrict__ desc,
                     const int64_t *__restrict__ boff,
                     int32_t *__restrict__ out) {
  __shared__ uint32_t tmp[kBlock / 64];
  // A block without edges has nothing to write (the scan is block-local).
  if (boff[blockIdx.x + 1] == boff[blockIdx.x]) return;
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  LinkSets ls{};
  uint32_t lc = 0, uc = 0;
  if (v < X * Y * Z) {
    ls = link_sets(f, X, Y, Z, v);
    lc = kLink.ncomp[ls.lower];
    uc = kLink.ncomp[ls.upper];
  }
  const uint32_t c = edge_count(lc, uc);
  uint32_t tot = 0;
  const uint32_t ex = block_scan16(c, tmp, &tot);
  if (c)
    egraph_emit(ls, v, X, X * Y, lc, uc, asc, desc, out,
                boff[blockIdx.x] + ex);
}

// Planes per walk: 16 share the two extra planes and the staged table well;
// four where the grid would not give each CU four blocks.
Walk make_walk(const float *f, const int64_t *dims, unsigned *blocks) {
  Walk w;
  w.f = f;
  w.X = (uint32_t)dims[0];
  w.Y = (uint32_t)dims[1];
  w.Z = (uint32_t)dims[2];
  w.XY = w.X * w.Y;
  w.runs = (w.XY + 63) / 64;
  w.pb = (w.XY + kWalkThreads - 1) / kWalkThreads;
  const uint64_t big = (uint64_t)w.pb * ((w.Z + 15) / 16);
  w.zc = big >= 1024 ? 16 : 4;
  *blocks = w.pb * ((w.Z + w.zc - 1) / w.zc);
  return w;
}

// The walk is for planes that fill a good part of its blocks (kWalkThreads
// positions each) and for more than one of them: a block of a narrow plane
// works, and stages its table, for few vertices, and a single plane is walked
// with two neighbour planes that are not there.  Critical points of 4.2M
// vertices, a vertex per thread / walked: planes of 8x8 positions 45 / 68 us,
// 12x10 44 / 50, 140x1 44 / 48, 18x9 45 / 46, 16x12 45 / 44, 16x16 44 / 39, 64x64
// 45 / 35; 1M vertices in a row 32 / 685; 4096x4096x1 99 / 110, 2048x2048x2
// 63 / 54.  (A walk of the narrowest planes would also be of more threads than a
// launch takes, 2^32, from Z = 2^27 on.)
bool walk_suits(const Walk &w) { return w.XY >= 192 && w.Z > 1; }

}  // namespace

int critical_points_run(msc_ctx *ctx, const float *field, const int64_t *dims,
                        uint8_t *code, hipStream_t s) {
  const int64_t N = dims[0] * dims[1] * dims[2];
  unsigned nb = 0;
  const Walk w = make_walk(field, dims, &nb);
  MSC_TRY(clear_counters(ctx, s));
  MSC_PHASE(ctx, s, "critical", 5.0 * N,
            (!walk_suits(w)
                 ? k_critical_small<<<grid_for(N), kBlock, 0, s>>>(
                       field, dims[0], dims[1], dims[2], code, ctx->dctr)
             : w.zc == 16
                 ? k_critical<16><<<nb, kWalkThreads, 0, s>>>(w, code, ctx->dctr)
                 : k_critical<4><<<nb, kWalkThreads, 0, s>>>(w, code,
                                                             ctx->dctr)));
  MSC_TRY(read_counters(ctx, s));
  if (ctx->hctr[kCtrNaN]) return MSC_ENAN;
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = N;
  return MSC_OK;
}

int extremum_graph_run(msc_ctx *ctx, const float *field, const int64_t *dims,
                       const int32_t *asc, const int32_t *desc, int32_t *edges,
                       int64_t capacity, int64_t *count, hipStream_t s) {
  const int64_t X = dims[0], Y = dims[1], Z = dims[2], N = X * Y * Z;
  unsigned wb = 0;
  const Walk w = make_walk(field, dims, &wb);
  auto need = [](int64_t nc, bool marked) {
    const int64_t nsb = (nc + kScan - 1) / kScan;
    return align256(nc * 4) + align256((nc + 1) * 8) + align256(nsb * 8 + 8) +
           (marked ? align256(nc * 8) : 0) + 4096;
  };
  const int64_t nb = (N + kBlock - 1) / kBlock;
  const int64_t runs = (int64_t)w.runs * Z;
  const bool marked = w.XY >= 64 && !(ctx->ws.external &&
                                      ctx->ws.bytes < need(runs, true));
  // Edge counts per run, or per block of 256 vertices.
  const int64_t nc = marked ? runs : nb;
  MSC_TRY(reserve(ctx, ctx->ws, need(nc, marked)));
  Carver cv(ctx->ws);
  uint32_t *cnt = cv.take<uint32_t>(nc);
  int64_t *off = cv.take<int64_t>(nc + 1);
  uint64_t *bsum = cv.take<uint64_t>((nc + kScan - 1) / kScan + 1);
  unsigned long long *marks =
      marked ? cv.take<unsigned long long>(nc) : nullptr;
  MSC_TRY(clear_counters(ctx, s));
  MSC_PHASE(
      ctx, s, "egraph_count", 4.0 * N,
      (marked && w.zc == 16
           ? k_egraph_mark<16><<<wb, kWalkThreads, 0, s>>>(w, marks, cnt,
                                                           ctx->dctr)
       : marked ? k_egraph_mark<4><<<wb, kWalkThreads, 0, s>>>(w, marks, cnt,
                                                               ctx->dctr)
                : k_egraph_count_small<<<(unsigned)nb, kBlock, 0, s>>>(
                    field, X, Y, Z, cnt, ctx->dctr),
       scan64(ctx, cnt, nc, off, bsum, s)));
  MSC_TRY(read_counters(ctx, s, off + nc));
  if (ctx->hctr[kCtrNaN]) return MSC_ENAN;
  const int64_t total = (int64_t)ctx->hctr[kCtrExtra];
  *count = total;
  if (edges && capacity >= total && total > 0) {
    // Runs per wave (see k_egraph_write).
    const int64_t least = std::max<int64_t>(1, std::min<int64_t>(4, nc / 4096)),
                  fill = std::min<int64_t>(30, 64 * nc / total) | 1;
    const int K = (int)std::max(least, fill);
    MSC_PHASE(ctx, s, "egraph_write", 4.0 * N + 12.0 * total,
              (marked ? k_egraph_write<<<grid64((nc + K - 1) / K * 64, kBlock),
                                         kBlock, kBlock * K * 2, s>>>(
                            w, (uint64_t)nc, K, marks, off, asc, desc, edges)
                      : k_egraph_write_small<<<(unsigned)nb, kBlock, 0, s>>>(
                            field, X, Y, Z, asc, desc, off, edges)));
    MSC_TRY(read_counters(ctx, s));
  }
  ctx->stats = msc_stats{};
  ctx->stats.n_vertices = N;
  return MSC_OK;
}

}  // namespace msc
