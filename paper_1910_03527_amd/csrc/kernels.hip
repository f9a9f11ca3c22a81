// HIP kernels of the MBE-FCI hot path for gfx950 (CDNA4), all FP64.
//
// One translation unit holds every kernel so that the binomial table lives in
// a single __constant__ object.  Launchers at the bottom are the only symbols
// the host runtime calls (declared in launch.h).
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace mbefci {

// ----------------------------------------------------------------- binomials
struct BinomTable {
  int64_t v[kBinom][kBinom];
};
constexpr BinomTable make_binom() {
  BinomTable t{};
  for (int n = 0; n < kBinom; ++n) {
    t.v[n][0] = 1;
    for (int k = 1; k <= n; ++k) t.v[n][k] = t.v[n - 1][k - 1] + (k <= n - 1 ? t.v[n - 1][k] : 0);
  }
  return t;
}
__constant__ BinomTable c_binom = make_binom();

__device__ inline int64_t binom(int n, int k) {
  return (n < 0 || k < 0 || k > n) ? 0 : c_binom.v[n][k];
}

// Address of a string (bitmask, ascending-integer order of all strings with
// the same popcount): combinatorial number system sum_j C(o_j, j), o_j the
// j-th occupied orbital (1-based j) in ascending order.
__device__ inline int64_t string_addr(uint64_t mask) {
  int64_t a = 0;
  int j = 1;
  while (mask) {
    int o = __builtin_ctzll(mask);
    a += binom(o, j++);
    mask &= mask - 1;
  }
  return a;
}

// Inverse of string_addr for strings of ne electrons.
__device__ inline uint64_t string_unrank(int64_t r, int n, int ne) {
  uint64_t mask = 0;
  int o = n - 1;
  for (int j = ne; j >= 1; --j) {
    while (binom(o, j) > r) --o;
    mask |= (uint64_t)1 << o;
    r -= binom(o, j);
    --o;
  }
  return mask;
}

// Lexicographic rank / unrank of a sorted k-combination of {0..N-1}.
__device__ inline int64_t comb_lex_rank(const int* c, int k, int N) {
  int64_t r = 0;
  int prev = -1;
  for (int i = 0; i < k; ++i) {
    for (int j = prev + 1; j < c[i]; ++j) r += binom(N - 1 - j, k - 1 - i);
    prev = c[i];
  }
  return r;
}
__device__ inline void comb_lex_unrank(int64_t r, int k, int N, int* c) {
  int j = 0;
  for (int i = 0; i < k; ++i) {
    while (true) {
      int64_t b = binom(N - 1 - j, k - 1 - i);
      if (r < b) break;
      r -= b;
      ++j;
    }
    c[i] = j++;
  }
}

// ------------------------------------------------- strings and link tables
__global__ void k_strings(int n, int ne, int64_t N, uint64_t* out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) out[i] = string_unrank(i, n, ne);
}

// One thread per string I: its single-excitation links E_pq|I> = s|J> in the
// canonical order (diagonal entries first, then q in I ascending, p not in I
// ascending).  The sign is (-1)^(number of occupied orbitals strictly between
// p and q), the parity of a+_p a_q acting on the occupation-number vector.
// abi4 lists (p, q, J, s).  The packed tables are the sigma gather's; the
// link-major copy packedT orders each string's links by ascending pair field
// (a string's off-diagonal links have distinct pairs, as have its diagonal
// ones): at link step l the lanes of a wave then read nearby rows of G's row
// block, which the L1 and L2 serve far better than the canonical order's
// spread.
__global__ void k_links(int n, int ne, int64_t N, uint32_t* packed, uint32_t* packedT,
                        int32_t* abi4) {
  constexpr int kSortMax = kMaxActive * (kMaxActive / 2 + 1);  // links of a CASCI string
  int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= N) return;
  const int L = ne * (n - ne + 1);
  const bool sortT = packedT && L <= kSortMax;
  uint32_t vs[kSortMax];
  uint64_t m = string_unrank(I, n, ne);
  int idx = 0;
  auto put = [&](uint32_t v) {
    if (packed) packed[I * L + idx] = v;
    if (sortT) vs[idx] = v;
    else if (packedT) packedT[idx * N + I] = v;
  };
  for (int o = 0; o < n; ++o)
    if (m >> o & 1) {
      put(pack_link((int)I, pair_index(o, o), 1));
      if (abi4) {
        int32_t* e = abi4 + (I * L + idx) * 4;
        e[0] = o; e[1] = o; e[2] = (int32_t)I; e[3] = 1;
      }
      ++idx;
    }
  for (int q = 0; q < n; ++q) {
    if (!(m >> q & 1)) continue;
    for (int p = 0; p < n; ++p) {
      if (m >> p & 1) continue;
      uint64_t r = (m & ~((uint64_t)1 << q)) | ((uint64_t)1 << p);
      int lo = p < q ? p : q, hi = p < q ? q : p;
      uint64_t between = (((uint64_t)1 << hi) - 1) & ~((((uint64_t)1 << lo) << 1) - 1);
      int sign = (__builtin_popcountll(m & between) & 1) ? -1 : 1;
      int64_t J = string_addr(r);
      put(pack_link((int)J, pair_index(hi, lo), sign));
      if (abi4) {
        int32_t* e = abi4 + (I * L + idx) * 4;
        e[0] = p; e[1] = q; e[2] = (int32_t)J; e[3] = sign;
      }
      ++idx;
    }
  }
  if (sortT)  // links in ascending pair field (distinct within a string)
    for (int a = 0; a < L; ++a) {
      int rank = 0;
      for (int b = 0; b < L; ++b) rank += link_pair(vs[b]) < link_pair(vs[a]);
      packedT[rank * N + I] = vs[a];
    }
}

// One thread per string K: for every orbital pair a >= b the non-vanishing
// member of {E_ab K, E_ba K} (see pack_pair_entry).
__global__ void k_pair_table(int n, int ne, int64_t N, int32_t* out, int32_t* outT) {
  int64_t K = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (K >= N) return;
  const int npair = n * (n + 1) / 2;
  const uint64_t m = string_unrank(K, n, ne);
  int32_t* row = out + K * npair;
  for (int a = 0; a < n; ++a)
    for (int b = 0; b <= a; ++b) {
      int32_t v = 0;
      const bool ia = m >> a & 1, ib = m >> b & 1;
      if (a == b) {
        if (ia) v = pack_pair_entry((int)K, 1);
      } else if (ia != ib) {
        // move the electron from the occupied one of (a, b) to the empty one
        const int q = ia ? a : b, p = ia ? b : a;
        const uint64_t r = (m & ~((uint64_t)1 << q)) | ((uint64_t)1 << p);
        const uint64_t between = (((uint64_t)1 << a) - 1) & ~((((uint64_t)1 << b) << 1) - 1);
        const int sign = (__builtin_popcountll(m & between) & 1) ? -1 : 1;
        v = pack_pair_entry((int)string_addr(r), sign);
      }
      row[a * (a + 1) / 2 + b] = v;
      outT[(int64_t)(a * (a + 1) / 2 + b) * N + K] = v;
    }
}

// ------------------------------------------------------- Hamiltonian set-up
// Frozen-core fold of the full-space Hamiltonian onto the active set A of one
// CASCI (frozen F = O \ A doubly occupied, all other orbitals deleted):
//   E_core = e_const + sum_{i in F} 2 h_ii + sum_{i,j in F} [2(ii|jj) - (ij|ji)]
//   h_eff_tu = h_tu + sum_{i in F} [2(tu|ii) - (ti|iu)]
// and the pair-space contraction matrix used by sigma = H c:
//   k_pq = h_eff_pq - 1/2 sum_{r in A} (pr|rq)
//   W_{ab,cd} = 1/2 (ab|cd) + (k_ab d_cd + d_ab k_cd) / (2N),  a>=b, c>=d,
// N = number of active electrons (the number operator acts as N on the CASCI
// space, which folds the one-body term into the single contraction).
struct ActiveSet {
  int n, na;
  int act[kMaxActive];
  int nf;
  int frz[kMaxOrb];
};

__device__ void build_item_hamiltonian(const ActiveSet& s, int M, const double* __restrict__ h1,
                                       const double* __restrict__ eri, double e_const, int nel,
                                       ItemHam* ham, double* W, int kpad) {
  const int t = threadIdx.x, nt = blockDim.x;
  const int n = s.n;
  __shared__ double s_red[256];
  __shared__ double s_k[kMaxActive * kMaxActive];
  auto G = [&](int p, int q, int r, int u) -> double {
    return eri[(((size_t)p * M + q) * M + r) * M + u];
  };
  // frozen-core energy
  double e = 0.0;
  for (int x = t; x < s.nf * s.nf; x += nt) {
    int i = s.frz[x / s.nf], j = s.frz[x % s.nf];
    e += 2.0 * G(i, i, j, j) - G(i, j, j, i);
  }
  for (int x = t; x < s.nf; x += nt) e += 2.0 * h1[s.frz[x] * M + s.frz[x]];
  s_red[t] = e;
  __syncthreads();
  for (int w = nt / 2; w > 0; w >>= 1) {
    if (t < w) s_red[t] += s_red[t + w];
    __syncthreads();
  }
  if (t == 0) {
    ham->ecore = e_const + s_red[0];
    ham->eri = eri;
    ham->M = M;
    for (int i = 0; i < kMaxActive; ++i) ham->act[i] = i < n ? s.act[i] : 0;
  }
  // effective one-electron operator, Coulomb/exchange diagonals
  for (int x = t; x < n * n; x += nt) {
    int tt = x / n, uu = x % n;
    int p = s.act[tt], q = s.act[uu];
    double v = h1[p * M + q];
    for (int f = 0; f < s.nf; ++f) {
      int i = s.frz[f];
      v += 2.0 * G(p, q, i, i) - G(p, i, i, q);
    }
    ham->heff[tt * kMaxActive + uu] = v;
    ham->J[tt * kMaxActive + uu] = G(p, p, q, q);
    ham->K[tt * kMaxActive + uu] = G(p, q, q, p);
    double kv = v;
    for (int r = 0; r < n; ++r) kv -= 0.5 * G(p, s.act[r], s.act[r], q);
    s_k[tt * kMaxActive + uu] = kv;
  }
  __syncthreads();
  if (W) {
    const double inv2n = nel > 0 ? 0.5 / nel : 0.0;
    const int npair = n * (n + 1) / 2;
    __shared__ uint16_t s_pair[kMaxActive * (kMaxActive + 1) / 2];
    for (int x = t; x < n * n; x += nt) {
      const int a = x / n, b = x % n;
      if (b <= a) s_pair[a * (a + 1) / 2 + b] = (uint16_t)(a << 8 | b);
    }
    __syncthreads();
    // (several elements' loads in flight, pairs looked up: a single CASCI has one
    // block; 31 -> 17 us at 12 orbitals)
#pragma unroll 8
    for (int x = t; x < kpad * kpad; x += nt) {
      const int ab = x / kpad, cd = x % kpad;
      const int pab = s_pair[min(ab, npair - 1)], pcd = s_pair[min(cd, npair - 1)];
      const int a = pab >> 8, b = pab & 255, c = pcd >> 8, d = pcd & 255;
      const double g = G(s.act[a], s.act[b], s.act[c], s.act[d]);
      double v = 0.0;
      if (ab < npair && cd < npair) {
        v = 0.5 * g;
        if (c == d) v += inv2n * s_k[a * kMaxActive + b];
        if (a == b) v += inv2n * s_k[c * kMaxActive + d];
      }
      W[x] = v;
    }
  }
}

// whether sigma of this CASCI contracts all pairs (needs W): the others take
// k_sigma_operands
__device__ inline bool pair_matrix(const Item& I) {
  return I.ndet > 1 && (I.sym || I.n > kStringMax);
}

// One block per item: decode the tuple of bucket (order, nocc) from its index
// (lexicographic ranks of its occupied and virtual parts), form A = R u T and
// F = O \ A, and build the item's folded Hamiltonian and W.
__global__ void k_mbe_setup(MbeSpaces sp, const BucketDev* __restrict__ buckets, int nbucket,
                            const Item* __restrict__ items, const double* __restrict__ h1,
                            const double* __restrict__ eri, double e_const, ItemHam* hams,
                            double* warena, int32_t* tuple_pos, int max_order,
                            int32_t* act_out) {
  const int it = blockIdx.x;
  __shared__ ActiveSet s;
  if (threadIdx.x == 0) {
    int b = 0;
    while (b + 1 < nbucket && buckets[b + 1].item0 <= it) ++b;
    const BucketDev bk = buckets[b];
    int64_t local = it - bk.item0;
    int nv = bk.order - bk.nocc;
    int64_t cv = binom(sp.nXv, nv);
    int64_t ro = local / cv, rv = local % cv;
    int co[kMaxActive], cvv[kMaxActive];
    comb_lex_unrank(ro, bk.nocc, sp.nXo, co);
    comb_lex_unrank(rv, nv, sp.nXv, cvv);
    // active set: merge R, Xo[co], Xv[cvv] (all disjoint), sorted ascending
    int tmp[kMaxActive];
    int nt = 0;
    for (int i = 0; i < sp.nR; ++i) tmp[nt++] = sp.R[i];
    for (int i = 0; i < bk.nocc; ++i) tmp[nt++] = sp.Xo[co[i]];
    for (int i = 0; i < nv; ++i) tmp[nt++] = sp.Xv[cvv[i]];
    for (int i = 1; i < nt; ++i) {
      int v = tmp[i], j = i - 1;
      while (j >= 0 && tmp[j] > v) { tmp[j + 1] = tmp[j]; --j; }
      tmp[j + 1] = v;
    }
    s.n = nt;
    for (int i = 0; i < nt; ++i) s.act[i] = tmp[i];
    s.nf = 0;
    for (int i = 0; i < sp.nO; ++i) {
      int o = sp.O[i];
      bool in = false;
      for (int j = 0; j < nt; ++j) in |= (tmp[j] == o);
      if (!in) s.frz[s.nf++] = o;
    }
    s.na = sp.nocc_ref + bk.nocc;
    if (act_out)
      for (int i = 0; i < kMaxActive; ++i) act_out[it * kMaxActive + i] = i < nt ? tmp[i] : -1;
    if (tuple_pos) {
      // positions: occupied part (indices into Xo), then virtual part (into Xv)
      int32_t* tp = tuple_pos + (int64_t)it * (2 * max_order + 2);
      tp[0] = bk.nocc;
      tp[1] = nv;
      for (int i = 0; i < bk.nocc; ++i) tp[2 + i] = co[i];
      for (int i = 0; i < nv; ++i) tp[2 + bk.nocc + i] = cvv[i];
    }
  }
  __syncthreads();
  const Item& I = items[it];
  build_item_hamiltonian(s, sp.M, h1, eri, e_const, I.na + I.nb, &hams[I.ham],
                         pair_matrix(I) ? warena + I.woff : nullptr, I.kpad);
}

// Direct CASCI set-up: the whole given space is active (no frozen orbitals).
__global__ void k_casci_setup(int n, const double* const* h1s, const double* const* eris,
                              const double* ecores, const Item* __restrict__ items, ItemHam* hams,
                              double* warena) {
  const int it = blockIdx.x;
  __shared__ ActiveSet s;
  if (threadIdx.x == 0) {
    s.n = n;
    for (int i = 0; i < n; ++i) s.act[i] = i;
    s.nf = 0;
    s.na = items[it].na;
  }
  __syncthreads();
  const Item& I = items[it];
  build_item_hamiltonian(s, n, h1s[it], eris[it], ecores[it], I.na + I.nb, &hams[I.ham],
                         pair_matrix(I) ? warena + I.woff : nullptr, I.kpad);
}

// --------------------------------------------------------------- diagonal
// H_II - E_core = sum_{p in Ia u Ib} h_eff_pp + sum_{p<q in Ia} [(pp|qq)-(pq|qp)]
//               + same for Ib + sum_{p in Ia, q in Ib} (pp|qq)
__global__ void k_hdiag(const Item* __restrict__ items, const Work* __restrict__ work,
                        const ItemHam* __restrict__ hams, double* diag) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const int64_t K = (int64_t)wk.begin * blockDim.x + threadIdx.x;
  if (K >= I.ndet) return;
  const ItemHam& H = hams[I.ham];
  uint64_t ma, mb;
  det_strings(I, K, ma, mb);
  double e = 0.0;
  for (uint64_t x = ma; x; x &= x - 1) {
    int p = __builtin_ctzll(x);
    e += H.heff[p * kMaxActive + p];
    for (uint64_t y = x & (x - 1); y; y &= y - 1) {
      int q = __builtin_ctzll(y);
      e += H.J[p * kMaxActive + q] - H.K[p * kMaxActive + q];
    }
    for (uint64_t y = mb; y; y &= y - 1) e += H.J[p * kMaxActive + __builtin_ctzll(y)];
  }
  for (uint64_t x = mb; x; x &= x - 1) {
    int p = __builtin_ctzll(x);
    e += H.heff[p * kMaxActive + p];
    for (uint64_t y = x & (x - 1); y; y &= y - 1) {
      int q = __builtin_ctzll(y);
      e += H.J[p * kMaxActive + q] - H.K[p * kMaxActive + q];
    }
  }
  diag[I.off + K] = e;
}

// ------------------------------------------------------------------ sigma
// sigma = (H - E_core) c.  Above kStringMax orbitals by the Knowles-Handy /
// Olsen factorisation
//   D+_ab[K] = <K| E_ab + E_ba |c>   (a > b),   D+_aa[K] = <K|E_aa|c>
//   G = W D+                          (the only dense step: FP64 MFMA)
//   sigma_I = sum over links E_xy I = s K of s G_pair(x,y)[K]
// (steps 1+2 fused in k_sigma_dgemm_pairrows, D+ tile in LDS, step 3 in
// k_sigma_gather); up to kStringMax orbitals from string operators (below).
// All read the vector slot given by `slot` (>= 0: fixed slot, items with
// slot >= their guess count skip; -1: the item's newest).
typedef double double4_t __attribute__((ext_vector_type(4)));

__device__ inline int vec_slot(const DavState& st, int slot) {
  return slot >= 0 ? slot : st.m - 1;
}
// f(std::integral_constant<int, M>{}) with M = m for m = 0..8 (returns
// true), else nothing (returns false): the Davidson passes loop over the
// subspace vectors with M known at compile time, so the loop unrolls without
// a branch per vector and a thread issues all of its loads at once.  Larger
// subspaces take the passes' generic loops.
template <class F>
__device__ inline bool with_space(int m, F&& f) {
  switch (m) {
    case 0: f(std::integral_constant<int, 0>{}); return true;
    case 1: f(std::integral_constant<int, 1>{}); return true;
    case 2: f(std::integral_constant<int, 2>{}); return true;
    case 3: f(std::integral_constant<int, 3>{}); return true;
    case 4: f(std::integral_constant<int, 4>{}); return true;
    case 5: f(std::integral_constant<int, 5>{}); return true;
    case 6: f(std::integral_constant<int, 6>{}); return true;
    case 7: f(std::integral_constant<int, 7>{}); return true;
    case 8: f(std::integral_constant<int, 8>{}); return true;
    default: return false;
  }
}
__device__ inline bool item_active(const DavState& st, int slot) {
  if (st.conv) return false;
  return slot < 0 || slot < st.nguess;
}

// Matrix element <I|H - E_core|J> between two different determinants of the
// active space (Slater-Condon rules; strings are bit masks over the active
// orbitals, alpha string before beta string, each in ascending order).
__device__ inline int between_parity(uint64_t s, int p, int q) {
  const int lo = p < q ? p : q, hi = p < q ? q : p;
  const uint64_t m = (((uint64_t)1 << hi) - 1) & ~((((uint64_t)1 << lo) << 1) - 1);
  return __builtin_popcountll(s & m) & 1;
}
__device__ double sc_offdiag(const ItemHam& H, uint64_t ia, uint64_t ib, uint64_t ja,
                             uint64_t jb) {
  const uint64_t xa = ia ^ ja, xb = ib ^ jb;
  const int da = __builtin_popcountll(xa) >> 1, db = __builtin_popcountll(xb) >> 1;
  if (da + db > 2) return 0.0;
  const double* __restrict__ eri = H.eri;
  const int M = H.M;
  auto g = [&](int p, int q, int r, int s) -> double {
    return ldg(eri + (((int64_t)H.act[p] * M + H.act[q]) * M + H.act[r]) * M + H.act[s]);
  };
  if (da + db == 1) {
    // one excitation q -> p in the string of spin sigma
    const uint64_t is = da ? ia : ib, js = da ? ja : jb, jo = da ? jb : ja;
    const int p = __builtin_ctzll(is & ~js), q = __builtin_ctzll(js & ~is);
    // sum over the occupied r of (pq|rr) per string less (pr|rq) for the
    // string's own (r = q contributes zero); the loads don't wait for each
    // other, as they would under a loop over set bits
    double v = H.heff[p * kMaxActive + q];
    const int top = 64 - __builtin_clzll(js | jo);
    const int ap = H.act[p], aq = H.act[q];
    const double* __restrict__ epq = eri + ((int64_t)ap * M + aq) * M * M;
    const double* __restrict__ ep = eri + (int64_t)ap * M * M * M + aq;
    for (int r0 = 0; r0 < top; r0 += 5) {
      double c[5], x[5];
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        const int a = H.act[min(r0 + u, top - 1)];
        c[u] = ldg(epq + (int64_t)a * (M + 1));
        x[u] = ldg(ep + ((int64_t)a * M + a) * M);
      }
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        const bool in = r0 + u < top;
        if (in && (js >> (r0 + u) & 1)) v += c[u] - x[u];
        if (in && (jo >> (r0 + u) & 1)) v += c[u];
      }
    }
    return between_parity(js, p, q) ? -v : v;
  }
  if (da == 1 && db == 1) {
    const int p = __builtin_ctzll(ia & ~ja), q = __builtin_ctzll(ja & ~ia);
    const int r = __builtin_ctzll(ib & ~jb), s = __builtin_ctzll(jb & ~ib);
    const double v = g(p, q, r, s);
    return (between_parity(ja, p, q) ^ between_parity(jb, r, s)) ? -v : v;
  }
  // two excitations in one string: holes q1 < q2, particles p1 < p2;
  // I = E_p1q1 E_p2q2 J (up to the sign), element (p1 q1|p2 q2) - (p1 q2|p2 q1)
  const uint64_t is = da ? ia : ib, js = da ? ja : jb;
  uint64_t pp = is & ~js, hh = js & ~is;
  const int p1 = __builtin_ctzll(pp), p2 = 63 - __builtin_clzll(pp);
  const int q1 = __builtin_ctzll(hh), q2 = 63 - __builtin_clzll(hh);
  const uint64_t k = (js & ~((uint64_t)1 << q2)) | ((uint64_t)1 << p2);
  const int par = between_parity(js, p2, q2) ^ between_parity(k, p1, q1);
  const double v = g(p1, q1, p2, q2) - g(p1, q2, p2, q1);
  return par ? -v : v;
}

constexpr int64_t binom_c(int n, int k) {
  int64_t r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

// Active spaces of up to kStringMax orbitals: H - E_core splits into a part
// in the alpha string, a part in the beta string and the opposite-spin part,
//   sigma = Ha C + C Hb + sum_{pq,rs} (pq|rs) Ea_pq Eb_rs C     (C = [Na][Nb]),
// with Ha, Hb the Slater-Condon matrices of one spin's strings.  The first two
// are dense products (k_sigma_same_spin).  In the third the alpha operators of
// one string Ia are its links only (1 + na (n - na) of the n (n + 1) / 2 pairs,
// the occupied diagonal ones taken together), so
//   E[rs][Jb] = sum_{links kl of Ia} s_kl (rs|kl) C[Ja][Jb]
// is a dense product of half the depth of one over all pairs, its B operand
// is rows of C as they stand in memory, and sigma[Ia][Ib] is a sum of E over
// the links of Ib: E of one alpha string stays in LDS and nothing but C and
// sigma passes through HBM (k_sigma_dgemm).
//
// FP64 products use v_mfma_f64_4x4x4_4b_f64: four independent 4x4x4 blocks.
// Measured rates of independent chains: 70-74 TFLOP/s from one wave per SIMD
// on, against 33 (one wave per SIMD) to 47 TFLOP/s (four) for the 16x16x4
// form.  Lane l holds A[l%4][l/16] and B[l/16][l%4] of block (l/4)%4 and
// receives D[l/16][l%4].  A 16-row A operand (lane l: row l%16) meets every
// 4-column block of a 16-column B operand in four instructions, with A's
// blocks rotated by r = 0..3: instruction r then holds row
// 4 ((b - r) & 3) + l/16 of column l%16, b = (l/4)%4.
template <int R>
__device__ inline double rot_blocks(double x) {  // block b takes block (b - R) & 3
  if constexpr (R == 0) {
    return x;
  } else {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x120 + 4 * R, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x120 + 4 * R, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
  }
}
// Load at a byte offset of 32 bits from a uniform base (one address register).
template <class T>
__device__ inline T ldg_at(const void* base, uint32_t bytes) {
  return ldg((const T*)((const char*)base + bytes));
}
__device__ inline double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
__device__ inline double flip_sign(double x, uint32_t bit31) {
  return __hiloint2double(__double2hiint(x) ^ (int)(bit31 & 0x80000000u), __double2loint(x));
}

// Work unit of this block: runs of kXcdRun consecutive units go to one XCD
// (blocks are dealt to the eight XCDs in turn), so that a CASCI's C, integral
// rows and string Hamiltonians are fetched into few of the eight L2s.
__device__ inline int xcd_unit(int block, int n) {
  constexpr int kRun = 16, kXcds = 8;
  const int whole = n / (kRun * kXcds) * (kRun * kXcds);
  if (block >= whole) return block;
  const int x = block % kXcds, k = block / kXcds;
  return (k / kRun * kXcds + x) * kRun + k % kRun;
}

// Integral rows of k_sigma_dgemm, per CASCI [2 no + Na + 1][kp] (no =
// n (n-1) / 2 off-diagonal pairs, kp = npair rounded up to 4): column c is
// (.|c) for off-diagonal pair c < no (offdiag_index) and (.|kk) for c = no + k;
// rows kl and no + kl are (kl|c) and -(kl|c), for links of either sign, row
// 2 no + Ia the sum over the occupied orbitals of alpha string Ia of (kk|c), the
// last row zero.  Then Ha and, for unequal electron counts, Hb, [np + 1][np] with np
// = strings rounded up to 16 and zero padding: the off-diagonal part and, in
// the last row, the diagonal.
__global__ void __launch_bounds__(256) k_sigma_operands(const Item* __restrict__ items,
                                                        const ItemHam* __restrict__ hams,
                                                        double* __restrict__ warena) {
  const Item& I = items[blockIdx.x];
  if (I.ndet <= 1 || I.sym || I.n > kStringMax) return;
  const ItemHam& H = hams[I.ham];
  const int n = I.n, no = n * (n - 1) / 2, kp = string_kp(n);
  const double* __restrict__ eri = H.eri;
  const int M = H.M;
  auto g = [&](int p, int q, int r, int s) -> double {
    return ldg(eri + (((int64_t)H.act[p] * M + H.act[q]) * M + H.act[r]) * M + H.act[s]);
  };
  const int64_t nv = (int64_t)(2 * no + I.Na + 1) * kp;
  const int pa = (I.Na + 15) & ~15, pb = (I.Nb + 15) & ~15;
  const int64_t na2 = (int64_t)(pa + 1) * pa, nb2 = I.na != I.nb ? (int64_t)(pb + 1) * pb : 0;
  double* __restrict__ out = warena + I.woff;
  const int64_t step = (int64_t)gridDim.y * 256;
  for (int64_t x = (int64_t)blockIdx.y * 256 + threadIdx.x; x < nv + na2 + nb2; x += step) {
    double v = 0.0;
    if (x < nv) {
      const int row = (int)(x / kp), c = (int)(x % kp);
      int a = 0, b = 0;
      if (c < no) {
        a = 1;
        while ((a + 1) * a / 2 <= c) ++a;
        b = c - a * (a - 1) / 2;
      } else {
        a = b = c - no;
      }
      if (a < n) {
        if (row < 2 * no) {
          const int kl = row < no ? row : row - no;
          int k = 1;
          while ((k + 1) * k / 2 <= kl) ++k;
          v = g(k, kl - k * (k - 1) / 2, a, b);
          if (row >= no) v = -v;
        } else if (row < 2 * no + I.Na) {
          for (uint64_t m = I.strA[row - 2 * no]; m; m &= m - 1) {
            const int k = __builtin_ctzll(m);
            v += g(k, k, a, b);
          }
        }
      }
    } else {
      const bool beta = x >= nv + na2;
      const int64_t y = x - nv - (beta ? na2 : 0);
      const int np = beta ? pb : pa, N = beta ? I.Nb : I.Na;
      const int i = (int)(y / np), j = (int)(y % np);
      const uint64_t* str = beta ? I.strB : I.strA;
      if ((i < N || i == np) && j < N && i != j) {
        const uint64_t mj = str[j];
        if (i == np) {  // the diagonal
          for (uint64_t z = mj; z; z &= z - 1) {
            const int p = __builtin_ctzll(z);
            v += H.heff[p * kMaxActive + p];
            for (uint64_t w = z & (z - 1); w; w &= w - 1) {
              const int q = __builtin_ctzll(w);
              v += H.J[p * kMaxActive + q] - H.K[p * kMaxActive + q];
            }
          }
        } else {
          v = sc_offdiag(H, str[i], 0, mj, 0);
        }
      }
    }
    out[x] = v;
  }
}

// Link tables of k_sigma_dgemm (either may be null), one thread per string of
// ne electrons.
// alpha [N][ks] (ks = string_kslots): slot k is the address Ja (bits 0..9) and
// the signed integral row (bits 10..20) of one off-diagonal link, then the
// diagonal slot (own address, row 2 no + I), then zero-row slots.
// beta [entry pairs of pass 0, then of pass 1][N]: two 16-bit entries each,
// bits 0..14 the position of E[rs][Jb] in LDS (row in the pass times
// string_stride plus Jb), bit 15 the sign, links in ascending row order,
// diagonal pairs last, filled up with the position of a zero.
__global__ void k_string_links(int n, int ne, int64_t N, uint32_t* alpha, uint32_t* beta) {
  const int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= N) return;
  const uint64_t m = string_unrank(I, n, ne);
  const int no = n * (n - 1) / 2, ks = string_kslots(n, ne);
  const int S = string_stride(n), rp = string_rows(n);
  uint32_t* __restrict__ al = alpha ? alpha + I * ks : nullptr;
  int k = 0, pass = 0, cnt = 0, base = 0;
  uint32_t held = 0;
  auto put = [&](uint32_t e) {
    if (!beta) return;
    if (cnt & 1) beta[(int64_t)(base + cnt / 2) * N + I] = held | (e << 16);
    else held = e;
    ++cnt;
  };
  auto close = [&]() {  // fill the pass up to its entry count with zeros
    const int full = 2 * string_gpairs(n, pass);
    while (beta && cnt < full) put((uint32_t)(rp * S));
    base += full / 2;
    cnt = 0;
    ++pass;
  };
  auto link = [&](int r, uint32_t J, uint32_t neg) {  // rows ascend from call to call
    while (r >= (pass + 1) * rp) close();
    put((uint32_t)((r - pass * rp) * S) + J | (neg << 15));
  };
  for (int a = 1; a < n; ++a)
    for (int b = 0; b < a; ++b) {
      const int r = a * (a - 1) / 2 + b;
      const bool ia = m >> a & 1, ib = m >> b & 1;
      if (ia == ib) continue;
      const uint64_t o = (m ^ ((uint64_t)1 << a)) ^ ((uint64_t)1 << b);
      const uint64_t between = (((uint64_t)1 << a) - 1) & ~((((uint64_t)1 << b) << 1) - 1);
      const uint32_t neg = __builtin_popcountll(m & between) & 1;
      const uint32_t J = (uint32_t)string_addr(o);
      if (al) al[k++] = J | ((uint32_t)(r + (neg ? no : 0)) << 10);
      link(r, J, neg);
    }
  if (al) al[k++] = (uint32_t)I | ((uint32_t)(2 * no + I) << 10);
  while (al && k < ks) al[k++] = (uint32_t)I | ((uint32_t)(2 * no + N) << 10);
  for (int o = 0; o < n; ++o)
    if (m >> o & 1) link(no + o, (uint32_t)I, 0u);
  while (pass < string_passes(n)) close();
}

// sigma = Ha C + C Hb.  One wave per tile of 16 RB alpha x 16 CB beta strings,
// the first sum over Ja, then the second over Jb, each in chunks of 16 (four
// k-steps, the next chunk's operands loaded while one is multiplied).  Ha's
// and Hb's symmetry and C's layout give every operand whole 128-byte lines:
// in the second sum lane l takes four consecutive C[Ia][Jb] and the k order
// is permuted to match.  Bound by the FP64 matrix pipe (2 (Na + Nb) flops per
// determinant, operands from L2): 0.26 ms for Hubbard-16, 50 TFLOP/s.
// Where a plan has few tiles (1 x 1 then) a wave is one chain of loads, so
// three chunks are in flight: CAS(10,10) 31 -> 22 us, 24 CAS(9,9)s 18.5 ->
// 15.3 us against one.
typedef double double2u_t __attribute__((ext_vector_type(2), aligned(8)));
typedef double double2_t __attribute__((ext_vector_type(2)));
template <int RB, int CB>
__global__ void __launch_bounds__(256, 2) k_sigma_same_spin(
    const Item* __restrict__ items, const Work* __restrict__ work, int nwork,
    const double* __restrict__ warena, const double* __restrict__ V, int64_t ntot,
    double* __restrict__ Sarena, const DavState* __restrict__ st, int slot) {
  const int unit = __builtin_amdgcn_readfirstlane(
      4 * xcd_unit((int)blockIdx.x, (int)gridDim.x) + (int)(threadIdx.x >> 6));
  if (unit >= nwork) return;
  const Work wk = work[unit];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (!item_active(S, slot)) return;
  const int vs = vec_slot(S, slot);
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int Na = I.Na, Nb = I.Nb;
  const int pa = (Na + 15) & ~15, pb = (Nb + 15) & ~15;
  const double* __restrict__ c = V + (int64_t)vs * ntot + I.off;
  const double* __restrict__ Ha = warena + I.woff +
                                  (int64_t)(I.n * (I.n - 1) + Na + 1) * string_kp(I.n);
  const double* __restrict__ Hb = I.na != I.nb ? Ha + (int64_t)(pa + 1) * pa : Ha;
  const int r0 = wk.begin * 16 * RB, c0 = wk.end * 16 * CB;  // first alpha, beta string
  int ia[RB], jb[CB];
#pragma unroll
  for (int r = 0; r < RB; ++r) ia[r] = min(r0 + 16 * r + li, Na - 1);
#pragma unroll
  for (int q = 0; q < CB; ++q) jb[q] = min(c0 + 16 * q + li, Nb - 1);
  double acc[RB][CB][4];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int q = 0; q < CB; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[r][q][v] = 0.0;
  constexpr int DEPTH = RB * CB == 1 ? 4 : 2;  // chunks in flight
  double A[DEPTH][RB][4], B[DEPTH][CB][4];
  auto load1 = [&](int k0, double (&a)[RB][4], double (&b)[CB][4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ja = k0 + 4 * j + lk;          // < pa
      const int jc = min(ja, Na - 1);          // Ha's rows beyond Na are zero
#pragma unroll
      for (int r = 0; r < RB; ++r) a[r][j] = ldg(Ha + ja * pa + ia[r]);
#pragma unroll
      for (int q = 0; q < CB; ++q) b[q][j] = ldg(c + jc * Nb + jb[q]);
    }
  };
  auto load2 = [&](int k0, double (&a)[RB][4], double (&b)[CB][4]) {
    const int j0 = k0 + 4 * lk;  // this lane's four Jb (< pb)
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const double* __restrict__ row = c + ia[r] * Nb;
      if (k0 + 16 <= Nb) {  // uniform
        const double2u_t x = ldg((const double2u_t*)(row + j0)),
                         y = ldg((const double2u_t*)(row + j0 + 2));
        a[r][0] = x[0], a[r][1] = x[1], a[r][2] = y[0], a[r][3] = y[1];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) a[r][j] = ldg(row + min(j0 + j, Nb - 1));
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int q = 0; q < CB; ++q) b[q][j] = ldg(Hb + (j0 + j) * pb + jb[q]);
  };
  auto multiply = [&](const double (&a)[RB][4], const double (&b)[CB][4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const double a1 = rot_blocks<1>(a[r][j]), a2 = rot_blocks<2>(a[r][j]),
                     a3 = rot_blocks<3>(a[r][j]);
#pragma unroll
        for (int q = 0; q < CB; ++q) {
          acc[r][q][0] = mfma4(a[r][j], b[q][j], acc[r][q][0]);
          acc[r][q][1] = mfma4(a1, b[q][j], acc[r][q][1]);
          acc[r][q][2] = mfma4(a2, b[q][j], acc[r][q][2]);
          acc[r][q][3] = mfma4(a3, b[q][j], acc[r][q][3]);
        }
      }
  };
  const int n1 = pa / 16, n2 = pb / 16;
  if constexpr (DEPTH > 2) {
    // either sum's chunk by the same loads, never under a branch (the compiler
    // would wait for every load in flight where the paths meet)
    auto load = [&](int k, double (&a)[RB][4], double (&b)[CB][4]) {
      const bool one = k < n1;  // uniform
      const int k0 = 16 * (one ? k : min(k, n1 + n2 - 1) - n1);
      const double* __restrict__ pa_ = one ? Ha : c;
      const double* __restrict__ pb_ = one ? c : Hb;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int j1 = k0 + 4 * j + lk, j2 = k0 + 4 * lk + j;
        a[0][j] = ldg(pa_ + (one ? j1 * pa + ia[0] : ia[0] * Nb + min(j2, Nb - 1)));
        b[0][j] = ldg(pb_ + (one ? min(j1, Na - 1) * Nb : j2 * pb) + jb[0]);
      }
    };
#pragma unroll
    for (int d = 0; d + 1 < DEPTH; ++d) load(d, A[d], B[d]);
    for (int k = 0; k < n1 + n2; k += DEPTH) {
#pragma unroll
      for (int h = 0; h < DEPTH; ++h) {
        load(k + h + DEPTH - 1, A[(h + DEPTH - 1) % DEPTH], B[(h + DEPTH - 1) % DEPTH]);
        if (k + h < n1 + n2) multiply(A[h], B[h]);
      }
    }
  } else {
    load1(0, A[0], B[0]);
    for (int k = 0; k < n1 + n2; k += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (k + h < n1 + n2) {
          const int nx = k + h + 1;
          if (nx < n1) load1(16 * nx, A[1 - h], B[1 - h]);
          else if (nx < n1 + n2) load2(16 * (nx - n1), A[1 - h], B[1 - h]);
          multiply(A[h], B[h]);
        }
      }
    }
  }
  // instruction v of lane l is row 4 ((b - v) & 3) + l/16: put row block v
  // into register v, so that a store covers whole 128-byte row pieces
  // The diagonal, the largest terms, is added to the finished sums: at the
  // start or middle of a chain every later term would round against it.
  double* __restrict__ out = Sarena + (int64_t)vs * ntot + I.off;
  const bool b1 = lane & 4, b2 = lane & 8;
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const double db = ldg(Hb + pb * pb + jb[q]);
      const double* x = acc[r][q];
      const double t0 = b1 ? x[1] : x[0], t1 = b1 ? x[0] : x[3], t2 = b1 ? x[3] : x[2],
                   t3 = b1 ? x[2] : x[1];
      const double y[4] = {b2 ? t2 : t0, b2 ? t3 : t1, b2 ? t0 : t2, b2 ? t1 : t3};
      const int kb = c0 + 16 * q + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ka = r0 + 16 * r + 4 * v + lk;
        if (ka < Na && kb < Nb)
          out[ka * Nb + kb] = fma(ldg(Ha + pa * pa + ka) + db, ldg(c + ka * Nb + kb), y[v]);
      }
    }
}

// Opposite-spin part, added to the same-spin part in sigma.  A workgroup of
// WPS x SPW waves takes SPW alpha strings at a time, WPS waves each.  Per pass
// of string_rows rows of E: a wave takes the rows' A operand (the string's
// integral rows, staged in LDS) into registers, every group of 4 rows
// replicated over the four MFMA blocks, multiplies its 16-column blocks of C
// rows (registers, loaded during the last pass of the string before) and
// stores E; then thread Ib sums E over the links of beta string Ib.  Loads for
// the next pass and string are in flight under the products, and a second
// workgroup's products run under one's sums.  Every E element is one chain
// over the string's links in slot order and every sum has a fixed order:
// sigma does not depend on WPS or SPW.  Bound by the FP64 matrix pipe and the
// vector instructions of the sums, which share its issue.  Measured, sweep of
// Hubbard-16 (10 orbitals, 12.8 M determinants in all): 0.82 ms, 37 TFLOP/s of
// E products (45 issued); before, the contraction of all pairs and its gather
// took 1.92 + 1.07 ms.  Rotating A's blocks through DPP moves instead of
// replicating them costs 0.89 ms, loads under branches (each of which makes
// the compiler wait for every load in flight) 1.06 ms.
template <int NACT>
struct StringShape {
  static constexpr int NP = NACT * (NACT + 1) / 2, NO = NP - NACT;
  static constexpr int KP = string_kp(NACT), P = string_passes(NACT), RP = string_rows(NACT);
  static constexpr int S = string_stride(NACT);
  static constexpr int CMAX = (int)binom_c(NACT, NACT / 2);
  static constexpr int KS = (1 + (NACT / 2) * ((NACT + 1) / 2) + 3) / 4;  // most k-steps
  static constexpr int KS0 = KS > 2 ? KS - 2 : 1;  // the tables hold at least these
  static constexpr int groups(int p) { return ((p + 1) * RP <= KP ? RP : KP - p * RP) / 4; }
  static constexpr int gbefore(int p) {  // entry pairs of the passes before p
    int s = 0;
    for (int q = 0; q < p; ++q) s += string_gpairs(NACT, q);
    return s;
  }
};

// waves per SIMD to compile for: 256, 168 and 128 registers suffice without
// spills, except two waves per string of 10 orbitals (eight column blocks each)
constexpr int string_waves(int nact, int wps) {
  return nact == 10 && wps == 2 ? 1 : nact >= 9 ? 2 : nact == 8 ? 3 : 4;
}
template <int NACT, int WPS, int SPW>
__global__ void __launch_bounds__(64 * WPS * SPW, string_waves(NACT, WPS)) k_sigma_dgemm(
    const Item* __restrict__ items, const Work* __restrict__ work,
    const double* __restrict__ warena, const double* __restrict__ V, int64_t ntot,
    double* __restrict__ Sarena, const DavState* __restrict__ st, int slot) {
  using T = StringShape<NACT>;
  constexpr int S = T::S, P = T::P;
  constexpr int TPS = 64 * WPS;                       // threads per string
  constexpr int JPT = (T::CMAX + TPS - 1) / TPS;      // beta strings per thread
  constexpr int CPW = ((T::CMAX + 15) / 16 + WPS - 1) / WPS;  // column blocks per wave
  constexpr int ELDS = T::RP * S + 2;                 // E of a string, then a zero
  constexpr int RP2 = T::RP / 2;                      // 16-byte pieces of a row in a pass
  constexpr int PCS = (4 * T::KS * RP2 + TPS - 1) / TPS;  // pieces per thread, rounded up
  __shared__ double Es[SPW * ELDS];
  __shared__ __align__(16) double As[SPW * 2 * PCS * TPS];
  const Work wk = work[xcd_unit((int)blockIdx.x, (int)gridDim.x)];
  const Item& I = items[wk.item];
  const DavState& D = st[wk.item];
  if (!item_active(D, slot)) return;
  const int vs = vec_slot(D, slot);
  const int Nb = I.Nb;
  const double* __restrict__ c = V + (int64_t)vs * ntot + I.off;
  const double* __restrict__ W = warena + I.woff;
  double* __restrict__ out = Sarena + (int64_t)vs * ntot + I.off;
  const uint32_t* __restrict__ klink = I.klink;
  const uint32_t* __restrict__ glink = I.glink;

  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int sw = wave / WPS, wi = wave % WPS;  // string of this wave, wave of the string
  const int ts = (int)threadIdx.x - sw * TPS;
  double* __restrict__ E = Es + sw * ELDS;
  double* __restrict__ Al = As + sw * 2 * PCS * TPS;  // [slot][row of the pass]
  if (ts == 0) E[T::RP * S] = 0.0;  // where filled-up entries point
  auto sync = [&]() {
    if constexpr (WPS > 1) {
      __syncthreads();
    } else {  // the string belongs to this wave: LDS is in order within it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  const int ncb = (Nb + 15) >> 4;
  auto string_at = [&](int s) { return min(s + sw, wk.end - 1); };

  // Every global load below is unconditional (clamped addresses): a load
  // under a branch would make the compiler wait for all loads in flight.
  auto body = [&](auto ks) {
    constexpr int KS = decltype(ks)::value;  // k-steps of this item's strings
    // Links of one string: per lane those of its k-steps (rows of C), per
    // thread those whose integral rows it copies to LDS.
    uint32_t eb[KS], ep[PCS], ep0[PCS];
    auto load_links = [&](int ka) {
      const uint32_t* __restrict__ row = klink + ka * (4 * KS);
#pragma unroll
      for (int k = 0; k < KS; ++k) eb[k] = ldg_at<uint32_t>(row + 4 * k, 4u * (uint32_t)lk);
#pragma unroll
      for (int x = 0; x < PCS; ++x) ep[x] = ldg_at<uint32_t>(row, 4u * (uint32_t)min((ts + x * TPS) / RP2, 4 * KS - 1));
    };
    double B[CPW][KS];  // this wave's columns of the string's C rows
    auto load_b = [&](int cw) {
      const uint32_t col = 8 * (uint32_t)min((wi + cw * WPS) * 16 + li, Nb - 1);
#pragma unroll
      for (int k = 0; k < KS; ++k)
        B[cw][k] = ldg_at<double>(c, (eb[k] & 0x3FFu) * (uint32_t)(8 * Nb) + col);
    };
    double2_t pr[PCS];  // integral rows on their way to LDS
    auto load_rows = [&](int p, const uint32_t (&e)[PCS]) {
#pragma unroll
      for (int x = 0; x < PCS; ++x) {
        const uint32_t col = (uint32_t)min(p * T::RP + 2 * ((ts + x * TPS) % RP2), T::KP - 2);
        pr[x] = ldg_at<double2_t>(W, (((e[x] >> 10) & 0x7FFu) * (uint32_t)T::KP + col) * 8);
      }
    };
    auto store_rows = [&]() {
#pragma unroll
      for (int x = 0; x < PCS; ++x) *(double2_t*)(Al + 2 * (ts + x * TPS)) = pr[x];
    };
    load_links(string_at(wk.begin));
#pragma unroll
    for (int cw = 0; cw < CPW; ++cw) load_b(cw);
    load_rows(0, ep);
#pragma unroll
    for (int x = 0; x < PCS; ++x) ep0[x] = ep[x];
    store_rows();
    load_links(string_at(wk.begin + SPW));
    sync();

    for (int s0 = wk.begin; s0 < wk.end; s0 += SPW) {
      const int orow = string_at(s0) * Nb;
      double same[JPT], sum0[JPT], sum1[JPT];
#pragma unroll
      for (int j = 0; j < JPT; ++j) {
        same[j] = ldg(out + orow + min(ts + j * TPS, Nb - 1));  // added last: the larger part
        sum0[j] = sum1[j] = 0.0;
      }

      auto pass = [&](auto pc) {
        constexpr int p = decltype(pc)::value;
        constexpr bool last = p + 1 == P;
        constexpr int NG = T::groups(p);  // groups of 4 rows
        // the rows of the next pass, or of the next string's first
        if constexpr (last) load_rows(0, ep);
        else load_rows(p + 1, ep0);
        // link entries of this thread's beta strings in this pass
        constexpr int GN = string_gpairs(NACT, p);
        const uint32_t* __restrict__ gl = glink + T::gbefore(p) * Nb;
        uint32_t u[JPT][GN];
#pragma unroll
        for (int j = 0; j < JPT; ++j) {
          uint32_t kb = 4u * (uint32_t)min(ts + j * TPS, Nb - 1);
          asm volatile("" : "+v"(kb));  // keeps the addresses out of registers between passes
#pragma unroll
          for (int q = 0; q < GN; ++q) u[j][q] = ldg_at<uint32_t>(gl + q * Nb, kb);
        }
        double a[KS][NG];  // the four blocks of a lane group hold the same 4 rows
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
          for (int g = 0; g < NG; ++g)
            a[k][g] = Al[(4 * k + lk) * T::RP + 4 * g + (lane & 3)];
#pragma unroll
        for (int cw = 0; cw < CPW; ++cw) {
          const int cb = wi + cw * WPS;
          if (cb < ncb) {
            double acc[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = 0.0;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
#pragma unroll
              for (int g = 0; g < NG; ++g) acc[g] = mfma4(a[k][g], B[cw][k], acc[g]);
            }
            double* __restrict__ Ec = E + cb * 16 + li;
#pragma unroll
            for (int g = 0; g < NG; ++g) Ec[(4 * g + lk) * S] = acc[g];
          }
          if constexpr (last) {  // the next string's, into the registers just read
            __builtin_amdgcn_sched_barrier(0);
            load_b(cw);
          }
        }
        sync();
        store_rows();  // every wave has read this pass's rows
#pragma unroll
        for (int j = 0; j < JPT; ++j)
#pragma unroll
          for (int q = 0; q < GN; ++q) {
            sum0[j] += flip_sign(E[u[j][q] & 0x7FFFu], u[j][q] << 16);
            sum1[j] += flip_sign(E[(u[j][q] >> 16) & 0x7FFFu], u[j][q]);
          }
        sync();
      };
      pass(std::integral_constant<int, 0>{});
      if constexpr (P > 1) pass(std::integral_constant<int, 1>{});
      if constexpr (P > 2) pass(std::integral_constant<int, 2>{});
      if constexpr (P > 3) pass(std::integral_constant<int, 3>{});
      static_assert(P <= 4, "passes");
#pragma unroll
      for (int j = 0; j < JPT; ++j) {
        const int kb = ts + j * TPS;
        if (s0 + sw < wk.end && kb < Nb) out[orow + kb] = same[j] + (sum0[j] + sum1[j]);
      }
#pragma unroll
      for (int x = 0; x < PCS; ++x) ep0[x] = ep[x];
      load_links(string_at(s0 + 2 * SPW));
    }
  };
  const int nks = string_kslots(NACT, I.na) / 4;
  if (nks == T::KS) body(std::integral_constant<int, T::KS>{});
  else if (nks == T::KS - 1 && T::KS > T::KS0) body(std::integral_constant<int, (T::KS - 1 > T::KS0 ? T::KS - 1 : T::KS0)>{});
  else body(std::integral_constant<int, T::KS0>{});
}

// Above kStringMax orbitals: contraction G = W D+ over all pairs.  A tile is
// one alpha string Ka and TN consecutive beta strings; a workgroup keeps one
// beta block (TN strings) and walks down a range of alpha strings (tiles are
// numbered column-major: tile = block * Na + Ka).  A thread builds the same
// (pair, column) slots of D+ in every tile; their beta pair-table entries are
// loaded once per work unit into LDS.  Per tile the c row of Ka is staged in
// LDS.  The alpha half of a D+ entry is wave-uniform: a scalar pair-table load
// and a coalesced row segment of c.  D+ [pair][TN] (B operand) is staged in
// LDS, the wave's W rows (A operand) sit in registers.  G is stored
// [Ka][pair_index][Kb], rows g_stride(Nb) long; the gather adds all links.
// Workgroups of 512 threads (two waves per SIMD) for 11-12 orbitals, 1024
// (four per SIMD) for 13-14, since their LDS holds one or two workgroups per
// CU; with 1024 the waves split a tile's output blocks by row block and column
// half.
constexpr int dgemm_threads(int nact) { return nact >= 13 ? 1024 : 512; }

template <int NACT, int TN, int NT = dgemm_threads(NACT)>
__global__ void __launch_bounds__(NT) k_sigma_dgemm_pairrows(
    const Item* __restrict__ items, const Work* __restrict__ work,
    const double* __restrict__ warena, const double* __restrict__ V, int64_t ntot,
    double* __restrict__ Garena, const DavState* __restrict__ st, int slot) {
  constexpr int NP = NACT * (NACT + 1) / 2;
  constexpr int KPAD = (NP + 15) / 16 * 16;
  constexpr int KS = (NP + 3) / 4;       // MFMA k-steps (4 pair rows per step)
  constexpr int KR = KS * 4;             // D+ rows held in LDS (zero beyond NP)
  constexpr int NRB = KPAD / 16;         // 16-row blocks of G
  constexpr int NW = NT / 64;            // waves per workgroup
  constexpr int NCB = TN / 16;           // 16-column blocks per tile
  constexpr int NCG = (NW >= 16 && NCB % 2 == 0) ? 2 : 1;  // column groups of waves
  constexpr int NRG = NW / NCG;          // row groups of waves
  constexpr int NCBW = NCB / NCG;        // column blocks per wave
  constexpr int RBW = (NRB + NRG - 1) / NRG;  // row blocks per wave
  constexpr int NSUB = NT / TN;          // row groups of the D+ build
  constexpr int NPER = (NP + NSUB - 1) / NSUB;
  constexpr int LDT = TN + 1;            // padded LDS row (doubles)
  constexpr int CMAX = (int)binom_c(NACT, NACT / 2);  // largest string count for NACT
  constexpr int CPT = (CMAX + NT - 1) / NT;           // c-row doubles per thread
  constexpr int TPT = (NP * TN + NT - 1) / NT;        // beta-table entries per thread
  __shared__ double Ds[KR * LDT];
  __shared__ int32_t Tb[NP * TN];
  __shared__ double Cr[CMAX];

  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (!item_active(S, slot)) return;
  const int vs = vec_slot(S, slot);
  const double* __restrict__ c = V + (int64_t)vs * ntot + I.off;
  double* __restrict__ G = Garena + I.goff;
  const int Na = I.Na, Nb = I.Nb;
  const int32_t* __restrict__ pA = I.pairA;
  const int32_t* __restrict__ pB = I.pairB;

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int col = t % TN;
  const int sub = (TN >= 64) ? __builtin_amdgcn_readfirstlane(t / TN) : t / TN;

  const int blk = wk.begin / Na;          // every work unit stays inside one beta block
  const int Kb0 = blk * TN;
  const int Kb = Kb0 + col;
  const double keep = Kb < Nb ? 1.0 : 0.0;  // ragged end of the row: zero columns
  const int Kbc = Kb < Nb ? Kb : Nb - 1;
  const double* __restrict__ ca = c + Kbc;  // alpha source of D+: ca[Ja * Nb]

  // Row blocks rb = wrot + NRG r and column blocks cg NCBW .. of this wave.
  // When the 16-row blocks of G do not come in multiples of NRG some waves
  // have one block fewer; rotating the assignment by workgroup spreads those
  // idle slots over the SIMDs.
  const int cg = NCG == 1 ? 0 : wave / NRG;
  const int wrot = ((NCG == 1 ? wave : wave % NRG) + (int)blockIdx.x) % NRG;
  // W rows of this wave's row blocks, as MFMA A operands: lane l holds
  // W[rb*16 + l%16][ks*4 + l/16] (B operand: lane l holds D+[ks*4 + l/16][l%16])
  double wreg[RBW][KS];
  const double* __restrict__ W = warena + I.woff;
#pragma unroll
  for (int r = 0; r < RBW; ++r) {
    const int rb = wrot + NRG * r;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      wreg[r][ks] = (rb < NRB) ? ldg(W + (rb * 16 + (lane & 15)) * KPAD + ks * 4 + (lane >> 4))
                               : 0.0;
  }
  // This thread's beta pair-table entries: slot i is pair sub + NSUB i of
  // column col (x = t + NT i has x / TN = sub + NSUB i and x % TN = col),
  // the slots it writes in every tile's D+.  Then the zero padding rows of D+.
  static_assert(TPT == NPER, "one pair-table entry per D+ slot of a thread");
#pragma unroll
  for (int i = 0; i < NPER; ++i) {
    const int ab = sub + NSUB * i;
    if (ab < NP) Tb[t + NT * i] = ldg(pB + ab * Nb + Kbc);
  }
  for (int x = NP * LDT + t; x < KR * LDT; x += NT) Ds[x] = 0.0;

  // Software pipeline over the tiles of the work unit: the alpha pair-table
  // entries of tile i+1 are loaded while tile i builds D+, and the c row and
  // alpha-half values of tile i+1 while tile i runs its MFMAs.
  int32_t ea[NPER];   // alpha pair-table entries of the current tile
  double ga[NPER];    // c values they address (alpha half of D+)
  double cr[CPT];     // this thread's share of the c row Ka
  // The alpha entries are wave-uniform per row (scalar loads): with TN = 32
  // a wave covers the two rows 2*wave and 2*wave+1 of each row group.
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto load_entries = [&](int ka, int32_t (&e)[NPER]) {
    const int32_t* __restrict__ pa = pA + ka * NP;
#pragma unroll
    for (int i = 0; i < NPER; ++i) {
      if constexpr (TN >= 64) {
        const int ab = sub + NSUB * i;
        e[i] = ab < NP ? ldc(pa + ab) : 0;
      } else {
        static_assert(TN == 32, "tile width 32, 64 or 128");
        const int ab0 = 2 * wave_u + NSUB * i;
        const int32_t e0 = ab0 < NP ? ldc(pa + ab0) : 0;
        const int32_t e1 = ab0 + 1 < NP ? ldc(pa + ab0 + 1) : 0;
        e[i] = lane < 32 ? e0 : e1;
      }
    }
  };
  auto load_values = [&](int ka) {
#pragma unroll
    for (int i = 0; i < NPER; ++i) ga[i] = ea[i] ? ldg(ca + ((ea[i] >> 1) - 1) * Nb) : 0.0;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int x = t + NT * j;
      cr[j] = x < Nb ? ldg(c + ka * Nb + x) : 0.0;
    }
  };
  load_entries(wk.begin - blk * Na, ea);
  load_values(wk.begin - blk * Na);

  for (int tile = wk.begin; tile < wk.end; ++tile) {
    const int Ka = tile - blk * Na;              // uniform
    const bool more = tile + 1 < wk.end;
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (t + NT * j < Nb) Cr[t + NT * j] = cr[j];
    int32_t en[NPER];
    if (more) {
      load_entries(Ka + 1, en);
    } else {
#pragma unroll
      for (int i = 0; i < NPER; ++i) en[i] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NPER; ++i) {
      const int ab = sub + NSUB * i;
      if (ab < NP) {
        const int32_t e = Tb[t + NT * i];
        const int jb = e ? (e >> 1) - 1 : 0;
        const double fa = ea[i] ? ((ea[i] & 1) ? -keep : keep) : 0.0;
        const double fb = e ? ((e & 1) ? -keep : keep) : 0.0;
        Ds[ab * LDT + col] = fa * ga[i] + fb * Cr[jb];
      }
    }
    __syncthreads();
    if (more) {
#pragma unroll
      for (int i = 0; i < NPER; ++i) ea[i] = en[i];
      load_values(Ka + 1);
    }
#pragma unroll
    for (int r = 0; r < RBW; ++r) {
      const int rb = wrot + NRG * r;
      if (rb >= NRB) continue;
      double4_t acc[NCBW];
#pragma unroll
      for (int cb2 = 0; cb2 < NCBW; ++cb2) acc[cb2] = (double4_t){0.0, 0.0, 0.0, 0.0};
      // B operands double-buffered in registers: the LDS reads of k-step
      // ks+1 are issued before the MFMAs of k-step ks
      double bq[2][NCBW];
      const double* bbase = Ds + (lane >> 4) * LDT + cg * NCBW * 16 + (lane & 15);
#pragma unroll
      for (int cb2 = 0; cb2 < NCBW; ++cb2) bq[0][cb2] = bbase[cb2 * 16];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) {
#pragma unroll
          for (int cb2 = 0; cb2 < NCBW; ++cb2)
            bq[(ks + 1) & 1][cb2] = bbase[(ks + 1) * 4 * LDT + cb2 * 16];
        }
#pragma unroll
        for (int cb2 = 0; cb2 < NCBW; ++cb2)
          acc[cb2] = __builtin_amdgcn_mfma_f64_16x16x4f64(wreg[r][ks], bq[ks & 1][cb2], acc[cb2],
                                                          0, 0, 0);
      }
      // instruction order for the scheduler: the first B reads, then per
      // k-step the next step's B reads (0x100: LDS read) ahead of this
      // step's MFMAs (0x008)
      __builtin_amdgcn_sched_group_barrier(0x100, NCBW, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) __builtin_amdgcn_sched_group_barrier(0x100, NCBW, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NCBW, 0);
      }
      const int Gs = g_stride(Nb);  // row stride of G
      double* __restrict__ Grow = G + (int64_t)Ka * NP * Gs;
#pragma unroll
      for (int cb2 = 0; cb2 < NCBW; ++cb2) {
        const int Kc = Kb0 + (cg * NCBW + cb2) * 16 + (lane & 15);
        if (Kc < Gs) {  // the row's padding too (zero: D+ is zero there), whole lines
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            // gfx950 FP64 16x16x4 output layout: register v of lane l is
            // row l/16 + 4v, column l%16 of the 16x16 block
            // non-temporal: at 11-14 orbitals G (a 1-3 MB row block per
            // alpha string) streams through the caches without reuse before
            // the gather, and cached stores only evict c and the tables
            const int row = rb * 16 + (lane >> 4) + 4 * v;
            if (row < NP) __builtin_nontemporal_store(acc[cb2][v], &Grow[row * Gs + Kc]);
          }
        }
      }
    }
    // No barrier here: the next tile's Cr stores follow this tile's second
    // barrier (every D+ read of Cr is done), and its D+ stores follow the
    // next first barrier (every MFMA read of Ds is done).
  }
}

// sigma_I = sum_{links (x,y,J,s) of Ia} s G_xy[J, Ib] + sum_{links of Ib} s G_xy[Ia, J].
// One wave per 64-determinant segment of one alpha row (segments are
// row-aligned), so the alpha string and its links are wave-uniform (scalar
// loads) and the alpha-part reads of G are coalesced rows.  Work units run
// in reverse order: the contraction wrote G in unit order, so the part it
// wrote last, still in the last-level cache, is read first.
__global__ void __launch_bounds__(256) k_sigma_gather(const Item* __restrict__ items,
                                                      const Work* __restrict__ work,
                                                      const double* __restrict__ Garena,
                                                      double* __restrict__ Sarena, int64_t ntot,
                                                      const DavState* __restrict__ st, int slot) {
  const Work wk = work[gridDim.x - 1 - blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (!item_active(S, slot)) return;
  const int vs = vec_slot(S, slot);
  const int Nb = I.Nb;
  const int segs = (Nb + 63) >> 6;  // segments per alpha row
  const int seg = __builtin_amdgcn_readfirstlane(wk.begin * 4 + (threadIdx.x >> 6));
  if (seg >= wk.end) return;
  const int Ka = __builtin_amdgcn_readfirstlane(seg / segs);
  const int Kb = (seg % segs) * 64 + (threadIdx.x & 63);
  if (Kb >= Nb) return;
  const double* __restrict__ G = Garena + I.goff;
  const int Gs = g_stride(Nb);  // row stride of G
  const int La = I.La, Lb = I.Lb;
  double acc0 = 0.0, acc1 = 0.0;
  const int np = I.npair;  // rows of G per alpha string
  const uint32_t* __restrict__ la = I.linkA + Ka * La;
  const double* __restrict__ Gcol = G + Kb;  // G[(Ja * npair + pair) * Gs + Kb]
  int l = 0;
  for (; l + 3 < La; l += 4) {
    const uint32_t e0 = ldc(la + l), e1 = ldc(la + l + 1), e2 = ldc(la + l + 2), e3 = ldc(la + l + 3);
    const double g0 = ldg(Gcol + (int64_t)(link_addr(e0) * np + link_pair(e0)) * Gs);
    const double g1 = ldg(Gcol + (int64_t)(link_addr(e1) * np + link_pair(e1)) * Gs);
    const double g2 = ldg(Gcol + (int64_t)(link_addr(e2) * np + link_pair(e2)) * Gs);
    const double g3 = ldg(Gcol + (int64_t)(link_addr(e3) * np + link_pair(e3)) * Gs);
    acc0 += link_sign(e0) * g0 + link_sign(e2) * g2;
    acc1 += link_sign(e1) * g1 + link_sign(e3) * g3;
  }
  for (; l < La; ++l) {
    const uint32_t e0 = ldc(la + l);
    acc0 += link_sign(e0) * ldg(Gcol + (int64_t)(link_addr(e0) * np + link_pair(e0)) * Gs);
  }
  const uint32_t* __restrict__ lb = I.linkBT + Kb;               // link l of Kb: lb[l * Nb]
  const double* __restrict__ Grow = G + (int64_t)Ka * np * Gs;  // G[(Ka * npair + pair) * Gs + Jb]
  l = 0;
  for (; l + 3 < Lb; l += 4) {
    const uint32_t e0 = ldg(lb + l * Nb), e1 = ldg(lb + (l + 1) * Nb), e2 = ldg(lb + (l + 2) * Nb),
                   e3 = ldg(lb + (l + 3) * Nb);
    const double g0 = ldg(Grow + link_pair(e0) * Gs + link_addr(e0));
    const double g1 = ldg(Grow + link_pair(e1) * Gs + link_addr(e1));
    const double g2 = ldg(Grow + link_pair(e2) * Gs + link_addr(e2));
    const double g3 = ldg(Grow + link_pair(e3) * Gs + link_addr(e3));
    acc0 += link_sign(e0) * g0 + link_sign(e2) * g2;
    acc1 += link_sign(e1) * g1 + link_sign(e3) * g3;
  }
  for (; l < Lb; ++l) {
    const uint32_t e0 = ldg(lb + l * Nb);
    acc0 += link_sign(e0) * ldg(Grow + link_pair(e0) * Gs + link_addr(e0));
  }
  Sarena[(int64_t)vs * ntot + I.off + (int64_t)Ka * Nb + Kb] = acc0 + acc1;
}

// ------------------------------------------------------ input validation
// Finiteness and permutational symmetry of the MO integrals, on the device
// (no host copy of the M^4 tensor): each element is compared with its
// partners h_qp, and (qp|rs), (pq|sr), (rs|pq), to 1e-12 times the larger of
// 1 and the two magnitudes.  Bits of *flags (integer atomics): 1 h not finite,
// 2 h not symmetric, 4 eri not finite, 8 eri lacks the 8-fold symmetry.
__global__ void k_check_integrals(const double* __restrict__ h1, const double* __restrict__ eri,
                                  int M, int* flags) {
  const int64_t n1 = (int64_t)M * M, n2 = n1 * n1;
  int f = 0;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n1 + n2;
       x += (int64_t)gridDim.x * blockDim.x) {
    auto close = [](double a, double b) {
      const double sc = fmax(1.0, fmax(fabs(a), fabs(b)));
      return fabs(a - b) <= 1e-12 * sc;
    };
    if (x < n1) {
      const int p = (int)(x / M), q = (int)(x % M);
      const double a = h1[x];
      if (!isfinite(a)) f |= 1;
      else if (!close(a, h1[(int64_t)q * M + p])) f |= 2;
    } else {
      const int64_t y = x - n1;
      const int s = (int)(y % M), r = (int)(y / M % M), q = (int)(y / n1 % M), p = (int)(y / n1 / M);
      const double a = eri[y];
      auto at = [&](int i, int j, int k, int l) { return eri[(((int64_t)i * M + j) * M + k) * M + l]; };
      if (!isfinite(a)) f |= 4;
      else if (!close(a, at(q, p, r, s)) || !close(a, at(p, q, s, r)) || !close(a, at(r, s, p, q)))
        f |= 8;
    }
  }
  if (f) atomicOr(flags, f);
}

void launch_check_integrals(const double* h1, const double* eri, int M, int* flags,
                            hipStream_t s) {
  const int64_t n = (int64_t)M * M * (1 + (int64_t)M * M);
  int64_t b = (n + 255) / 256;
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_check_integrals, dim3((int)b), dim3(256), 0, s, h1, eri, M, flags);
}

// ------------------------------------------------- point-group blocked sigma
// The contraction of one pair class s on the determinants of irrep G^s:
// G_s = W_s D+_s on FP64 MFMA.  A work unit is (item, class s, alpha irrep
// a' of the irrep-G^s space) and a range of tiles of that block; a tile is
// one alpha string ka (local to irrep a') and TN consecutive beta strings of
// irrep b' = a'^G^s, numbered column-major (tile = block * nac[a'] + ka) so
// a unit stays inside one beta block.  D+ rows are the class's pairs,
// zero-padded to NPC.  The alpha half of a D+ entry reads c in CI block a'^s
// (beta irrep b', rows of nbc[b']), the beta half in block a' (rows of
// nbc[a'^G]).  Work.pad_ = s * 8 + a'.  Classes of up to 48 pairs take
// 64-column tiles with one 16-column block per wave (every wave busy however
// few row blocks the class has); larger ones 32-column tiles with row blocks
// dealt over the waves.
int sym_tile(int npc) { return npc <= 48 ? 64 : 32; }

template <int NPC, int TN>
__global__ void __launch_bounds__(256) k_sigma_sym_dgemm(
    const Item* __restrict__ items, const Work* __restrict__ work,
    const double* __restrict__ warena, const double* __restrict__ V, int64_t ntot,
    double* __restrict__ Garena, const DavState* __restrict__ st, int slot) {
  constexpr int KS = NPC / 4;       // MFMA k-steps
  constexpr int NRB = NPC / 16;     // 16-row blocks of G_s
  constexpr int NCB = TN / 16;
  constexpr bool COL = NCB == 4;    // wave w computes column block w, every row block
  constexpr int RBW = COL ? NRB : (NRB + 3) / 4;
  constexpr int LDT = TN + 1;
  __shared__ double Ds[NPC * LDT];
  __shared__ int32_t pl[NPC];       // class pair -> pair index (W row / column)

  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (!item_active(S, slot)) return;
  const SymInfo& Y = *I.sym;
  const int vs = vec_slot(S, slot);
  const double* __restrict__ c = V + (int64_t)vs * ntot + I.off;
  const int s = wk.pad_ >> 3, ap = wk.pad_ & 7;
  const int G = Y.wfn;
  const int bp = ap ^ G ^ s;          // beta irrep of the tile
  const int nps = Y.cls0[s + 1] - Y.cls0[s];
  const int j0 = Y.cls0[s];
  const int NA = Y.nac[ap], NB = Y.nbc[bp];
  const int NBa = Y.nbc[ap ^ G];      // row length of CI block a'
  const double* __restrict__ csrcA = c + Y.blk[ap ^ s];  // block a'^s: rows of NB
  const double* __restrict__ csrcB = c + Y.blk[ap];      // block a': rows of NBa
  const int32_t* __restrict__ pA = I.pairA + (int64_t)Y.na0[ap] * Y.npair + j0;
  const int32_t* __restrict__ pB = I.pairB + (int64_t)j0 * I.Nb + Y.nb0[bp];
  double* __restrict__ G_s = Garena + I.goff + Y.gofs[s][ap];
  const int kpad = I.kpad;
  const double* __restrict__ W = warena + I.woff;

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int i = t; i < NPC; i += 256) pl[i] = i < nps ? Y.pair_of[j0 + i] : -1;
  __syncthreads();
  const int wrot = (wave + (int)blockIdx.x) & 3;
  double wreg[RBW][KS];
#pragma unroll
  for (int r = 0; r < RBW; ++r) {
    const int rb = COL ? r : wrot + 4 * r;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int row = rb * 16 + (lane & 15), col = ks * 4 + (lane >> 4);
      wreg[r][ks] = (rb < NRB && row < nps && col < nps)
                        ? ldg(W + (int64_t)pl[row] * kpad + pl[col]) : 0.0;
    }
  }
  const int blk = wk.begin / NA;
  const int kb0 = blk * TN;
  // Classes of up to 32 pairs: this thread builds the D+ slots (class pair
  // sub + NSUB k, column col) of every tile of the unit; their beta
  // pair-table entries depend on the column only, so they are loaded once
  // per unit, and the alpha entries are wave-uniform per pair row (scalar
  // loads).  Larger classes build D+ element by element (registers for the
  // slots would cost them occupancy).
  constexpr bool SLOTS = NPC <= 32;
  constexpr int NSUB = 256 / TN;
  constexpr int NPER = SLOTS ? (NPC + NSUB - 1) / NSUB : 1;
  const int col = t % TN;
  const int sub = TN >= 64 ? __builtin_amdgcn_readfirstlane(t / TN) : t / TN;
  const int kb = kb0 + col;
  const bool live = kb < NB;
  const int kbc = live ? kb : NB - 1;
  int32_t eb[NPER];
  int32_t ea[NPER];
  double ga[NPER], gb[NPER];
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto load_tile = [&](int ka) {
    const int32_t* __restrict__ pa = pA + (int64_t)ka * Y.npair;
    const double* __restrict__ crow = csrcB + (int64_t)ka * NBa;
#pragma unroll
    for (int k = 0; k < NPER; ++k) {
      if constexpr (TN >= 64) {
        const int i = sub + NSUB * k;
        ea[k] = (i < nps) ? ldc(pa + i) : 0;
      } else {
        const int i0 = 2 * wave_u + NSUB * k;
        const int32_t e0 = i0 < nps ? ldc(pa + i0) : 0;
        const int32_t e1 = i0 + 1 < nps ? ldc(pa + i0 + 1) : 0;
        ea[k] = lane < 32 ? e0 : e1;
      }
      ga[k] = ea[k] ? ldg(csrcA + (int64_t)((ea[k] >> 1) - 1) * NB + kbc) : 0.0;
      gb[k] = eb[k] ? ldg(crow + ((eb[k] >> 1) - 1)) : 0.0;
    }
  };
  if constexpr (SLOTS) {
#pragma unroll
    for (int k = 0; k < NPER; ++k) {
      const int i = sub + NSUB * k;
      eb[k] = (i < nps && live) ? ldg(pB + (int64_t)i * I.Nb + kbc) : 0;
    }
  }
  for (int tile = wk.begin; tile < wk.end; ++tile) {
    const int ka = tile - blk * NA;
    // D+ tile [NPC][TN]: class pair i, column kb0 + col
    if constexpr (SLOTS) {
      load_tile(ka);
#pragma unroll
      for (int k = 0; k < NPER; ++k) {
        const int i = sub + NSUB * k;
        if (i < NPC) {
          const double fa = (ea[k] && live) ? ((ea[k] & 1) ? -1.0 : 1.0) : 0.0;
          const double fb = eb[k] ? ((eb[k] & 1) ? -1.0 : 1.0) : 0.0;
          Ds[i * LDT + col] = fa * ga[k] + fb * gb[k];
        }
      }
    } else {
      for (int x = t; x < NPC * TN; x += 256) {
        const int i = x / TN, cx = x % TN, kx = kb0 + cx;
        double v = 0.0;
        if (i < nps && kx < NB) {
          const int32_t e1 = ldg(pA + (int64_t)ka * Y.npair + i);
          if (e1) {
            const double cv = ldg(csrcA + (int64_t)((e1 >> 1) - 1) * NB + kx);
            v += (e1 & 1) ? -cv : cv;
          }
          const int32_t e2 = ldg(pB + (int64_t)i * I.Nb + kx);
          if (e2) {
            const double cv = ldg(csrcB + (int64_t)ka * NBa + ((e2 >> 1) - 1));
            v += (e2 & 1) ? -cv : cv;
          }
        }
        Ds[i * LDT + cx] = v;
      }
    }
    __syncthreads();
    // G rows are written with non-temporal stores: the class's G block is
    // not re-read before the gather (8 x CAS(14,14) in A_g: 59.8 -> 56.4 ms)
    double* __restrict__ Grows = G_s + (int64_t)ka * nps * NB;
    if constexpr (COL) {
      // this wave: columns kb0 + 16 wave .. + 15, every row block
      const double* bbase = Ds + (lane >> 4) * LDT + wave * 16 + (lane & 15);
      double4_t acc[NRB];
#pragma unroll
      for (int r = 0; r < NRB; ++r) acc[r] = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const double bv = bbase[ks * 4 * LDT];
#pragma unroll
        for (int r = 0; r < NRB; ++r)
          acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(wreg[r][ks], bv, acc[r], 0, 0, 0);
      }
      const int kc = kb0 + wave * 16 + (lane & 15);
      if (kc < NB) {
#pragma unroll
        for (int r = 0; r < NRB; ++r)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            // register v of lane l: row l/16 + 4v, column l%16 of the block
            const int row = r * 16 + (lane >> 4) + 4 * v;
            if (row < nps) __builtin_nontemporal_store(acc[r][v], &Grows[(int64_t)row * NB + kc]);
          }
      }
    } else {
#pragma unroll
      for (int r = 0; r < RBW; ++r) {
        const int rb = wrot + 4 * r;
        if (rb >= NRB) continue;
        double4_t acc[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[cb] = (double4_t){0.0, 0.0, 0.0, 0.0};
        const double* bbase = Ds + (lane >> 4) * LDT + (lane & 15);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(wreg[r][ks],
                                                           bbase[ks * 4 * LDT + cb * 16], acc[cb],
                                                           0, 0, 0);
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          const int kc = kb0 + cb * 16 + (lane & 15);
          if (kc < NB) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int row = rb * 16 + (lane >> 4) + 4 * v;
              if (row < nps) __builtin_nontemporal_store(acc[cb][v], &Grows[(int64_t)row * NB + kc]);
            }
          }
        }
      }
    }
    __syncthreads();  // every MFMA read of Ds is done before the next tile's build
  }
}

// sigma_I = sum over links of I of sign * G_s[K], blocked layout: one thread per
// determinant I = (a, ia, ib) of irrep G (b = a^G).  An alpha link of ia
// (class-sorted pair j of class s, string Ja local to irrep a^s) reads G_s in
// block a^s, row (Ja, j - cls0[s]), column ib; a beta link of ib (string Jb
// local to irrep b^s) reads G_s in block a, row (ia, j - cls0[s]), column Jb.
// The class tables are staged in LDS; beta links come from the link-major
// table linkBT [Lb][Nb] (consecutive threads read consecutive entries).
// Work units: 256 consecutive determinants of one item (Work.begin).
__global__ void __launch_bounds__(256) k_sigma_sym_gather(const Item* __restrict__ items,
                                                          const Work* __restrict__ work,
                                                          const double* __restrict__ Garena,
                                                          double* __restrict__ Sarena,
                                                          int64_t ntot,
                                                          const DavState* __restrict__ st,
                                                          int slot) {
  __shared__ int8_t cls_of[kMaxPair];
  __shared__ int32_t cls0[kIrreps + 1];
  __shared__ int32_t nbc[kIrreps];
  __shared__ int64_t gofs[kIrreps][kIrreps];
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (!item_active(S, slot)) return;  // uniform over the block (one item)
  const SymInfo& Y = *I.sym;
  const int t = threadIdx.x;
  for (int j = t; j < Y.npair; j += 256) cls_of[j] = Y.cls_of[j];
  if (t <= kIrreps) cls0[t] = Y.cls0[t];
  if (t < kIrreps) nbc[t] = Y.nbc[t];
  if (t < kIrreps * kIrreps) gofs[t >> 3][t & 7] = Y.gofs[t >> 3][t & 7];
  __syncthreads();
  const int64_t K = (int64_t)wk.begin * blockDim.x + t;
  if (K >= I.ndet) return;
  const int vs = vec_slot(S, slot);
  const int G = Y.wfn;
  int a = 0;
  while (a < kIrreps - 1 && K >= Y.blk[a + 1]) ++a;
  const int b = a ^ G;
  const int64_t loc = K - Y.blk[a];
  const int ia = (int)(loc / nbc[b]), ib = (int)(loc % nbc[b]);
  const double* __restrict__ Gi = Garena + I.goff;
  double acc0 = 0.0, acc1 = 0.0;
  const uint32_t* __restrict__ la = I.linkA + (int64_t)(Y.na0[a] + ia) * I.La;
  for (int l = 0; l < I.La; ++l) {
    const uint32_t e = ldg(la + l);
    const int j = link_pair(e), s = cls_of[j];
    const int c0 = cls0[s], nps = cls0[s + 1] - c0;
    acc0 += link_sign(e) * ldg(Gi + gofs[s][a ^ s] +
                               ((int64_t)link_addr(e) * nps + (j - c0)) * nbc[b] + ib);
  }
  const uint32_t* __restrict__ lb = I.linkBT + Y.nb0[b] + ib;  // link l: lb[l * Nb]
  for (int l = 0; l < I.Lb; ++l) {
    const uint32_t e = ldg(lb + (int64_t)l * I.Nb);
    const int j = link_pair(e), s = cls_of[j];
    const int c0 = cls0[s], nps = cls0[s + 1] - c0;
    acc1 += link_sign(e) * ldg(Gi + gofs[s][a] +
                               ((int64_t)ia * nps + (j - c0)) * nbc[b ^ s] + link_addr(e));
  }
  Sarena[(int64_t)vs * ntot + I.off + K] = acc0 + acc1;
}

// ---------------------------------------------------------------- Davidson
// Sum over the 16 lanes of a row, the same value in every lane of it: four DPP
// steps (a shuffle through the LDS crossbar takes several times as long).
template <int CTRL>
__device__ inline double dpp_move(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double row_sum(double x) {
#pragma clang fp contract(off)  // x may be a product: every lane has to round it
  x += dpp_move<0xB1>(x);   // quad_perm [1, 0, 3, 2]
  x += dpp_move<0x4E>(x);   // quad_perm [2, 3, 0, 1]
  x += dpp_move<0x141>(x);  // row_half_mirror
  x += dpp_move<0x140>(x);  // row_mirror
  return x;
}
__device__ inline double lane_value(double x, int lane) {  // lane: wave-uniform
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
  return __hiloint2double(hi, lo);
}
// Sum over the wave (all 64 lanes active), the same value in every lane.
__device__ inline double wave_sum64(double v) {
  v = row_sum(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Block-level fixed-order reduction of values per thread (256 threads): slots
// i < m and i >= fixed of v; the others are not written.
template <int NV>
__device__ inline void block_reduce_store(double (&v)[NV], int m, int fixed, double* out) {
  __shared__ double red[4][NV];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i)
    if (i < m || i >= fixed) {  // uniform
      const double x = wave_sum64(v[i]);
      if (lane == 0) red[wave][i] = x;
    }
  __syncthreads();
  for (int i = threadIdx.x; i < NV; i += blockDim.x)
    if (i < m || i >= fixed) out[i] = ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
  __syncthreads();
}

constexpr int kPart = kMaxSpace + 2;  // partial sums per chunk
constexpr int kChunk = 4096;          // elements per reduction chunk

// zero a vector slot range for the given items (fill kernel; graph safe)
__global__ void k_fill(double* p, int64_t n, double v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Dense guess vector: r_K = +-1/sqrt(ndet) with the sign taken from the top
// bit of a multiplicative hash of the address K.  It has no symmetry, so it
// carries weight in every spin and spatial symmetry sector of the
// determinant basis: with it in the first subspace the solver cannot be
// confined to a sector without the ground state (a closed-shell determinant,
// for example, is a pure singlet and never reaches a triplet ground state).
__device__ inline double hash_sign(int64_t K) {
  return (((uint64_t)K * 0x9E3779B97F4A7C15ull) >> 63) ? 1.0 : -1.0;
}

// Guess: the `nguess` lowest diagonal determinants (ties: lower address) as
// unit vectors in slots 0..g-1, and the dense vector orthogonalised against
// them in slot g.  One block per item.
__global__ void k_dav_guess(const Item* __restrict__ items, int ibase,
                            const double* __restrict__ diag, double* V, int64_t ntot, DavState* st,
                            int nguess) {
  const Item& I = items[ibase + blockIdx.x];
  DavState& S = st[ibase + blockIdx.x];
  const int t = threadIdx.x;
  constexpr int G = 8;
  double bv[G];
  int64_t bi[G];
  for (int g = 0; g < G; ++g) { bv[g] = 1e300; bi[g] = INT64_MAX; }
  const double* d = diag + I.off;
  for (int64_t K = t; K < I.ndet; K += blockDim.x) {
    double x = d[K];
    // insert (x, K) into the sorted list (value, then index)
    if (x < bv[G - 1] || (x == bv[G - 1] && K < bi[G - 1])) {
      int p = G - 1;
      while (p > 0 && (x < bv[p - 1] || (x == bv[p - 1] && K < bi[p - 1]))) {
        bv[p] = bv[p - 1]; bi[p] = bi[p - 1]; --p;
      }
      bv[p] = x; bi[p] = K;
    }
  }
  // g rounds of a block-wide argmin over the heads of the per-thread lists
  __shared__ double rv[256];
  __shared__ int64_t ri[256];
  __shared__ int rth[256];
  int g = nguess < G ? nguess : G;
  if (g > I.ndet) g = (int)I.ndet;
  __shared__ int64_t chosen[G];
  int head = 0;
  for (int k = 0; k < g; ++k) {
    rv[t] = head < G ? bv[head] : 1e300;
    ri[t] = head < G ? bi[head] : INT64_MAX;
    rth[t] = t;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (t < w) {
        const double v2 = rv[t + w];
        const int64_t i2 = ri[t + w];
        if (v2 < rv[t] || (v2 == rv[t] && i2 < ri[t])) {
          rv[t] = v2;
          ri[t] = i2;
          rth[t] = rth[t + w];
        }
      }
      __syncthreads();
    }
    if (t == rth[0]) ++head;
    if (t == 0) {
      V[(int64_t)k * ntot + I.off + ri[0]] = 1.0;
      chosen[k] = ri[0];
    }
    __syncthreads();
  }
  // dense vector minus its components on the chosen unit vectors
  const bool dense = I.ndet > g;
  if (dense) {
    const double sc = 1.0 / sqrt((double)(I.ndet - g));
    double* __restrict__ vr = V + (int64_t)g * ntot + I.off;
    for (int64_t K = t; K < I.ndet; K += blockDim.x) {
      bool hit = false;
      for (int j = 0; j < g; ++j) hit |= chosen[j] == K;
      vr[K] = hit ? 0.0 : hash_sign(K) * sc;
    }
  }
  if (t == 0) {
    S.m = 0;
    S.nguess = g + (dense ? 1 : 0);
    S.np = 0;
    S.onepass = 0;
    S.olsen = 0;
    S.iters = 0;
    S.status = 0;
    S.rnorm = 0.0;
    S.conv = 0;
    S.theta = 0.0;
    if (I.ndet == 1) {
      S.conv = 1;
      S.m = 1;
      S.theta = d[0];
    }
  }
}

// partial dots p_i = V_i . S_j over one chunk, for i < m (j = newest or `slot`)
__global__ void __launch_bounds__(256) k_dav_dots(const Item* __restrict__ items,
                                                  const Work* __restrict__ work,
                                                  const double* __restrict__ V,
                                                  const double* __restrict__ Sv, int64_t ntot,
                                                  const DavState* __restrict__ st, int slot,
                                                  double* part) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (!item_active(S, slot)) return;
  const int j = slot >= 0 ? slot : S.m - 1;
  const int m = j + 1;
  double acc[kMaxSpace];
#pragma unroll
  for (int i = 0; i < kMaxSpace; ++i) acc[i] = 0.0;
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  const double* sj = Sv + (int64_t)j * ntot + I.off;
  const bool unrolled = with_space(m, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      const double s = sj[e];
#pragma unroll
      for (int i = 0; i < M; ++i) acc[i] += V[(int64_t)i * ntot + I.off + e] * s;
    }
  });
  if (!unrolled) {
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      const double s = sj[e];
  #pragma unroll
      for (int i = 0; i < kMaxSpace; ++i)
        if (i < m) acc[i] += V[(int64_t)i * ntot + I.off + e] * s;
    }
  }
  block_reduce_store<kMaxSpace>(acc, m, kMaxSpace, part + (int64_t)wk.begin * kPart);
}

// Totals of an item's chunk partials by one wave: lane s < kPart returns slot s,
// summed over chunks g, g + 3, ... by the lanes of group g, then over g.
__device__ inline double wave_parts(const double* __restrict__ part, const Item& I) {
  const int lane = threadIdx.x & 63, s = lane % kPart, g = lane / kPart;
  const double* __restrict__ p = part + (int64_t)I.chunk0 * kPart + s;
  double v = 0.0;
  if (g < 3) {
    int c = g;
    for (; c + 21 < I.nchunk; c += 24) {  // eight loads in flight
      double x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = ldg(p + (int64_t)(c + 3 * q) * kPart);
#pragma unroll
      for (int q = 0; q < 8; ++q) v += x[q];
    }
    for (; c < I.nchunk; c += 3) v += ldg(p + (int64_t)c * kPart);
  }
  static_assert(3 * kPart <= 64, "three lane groups");
  const double v1 = __shfl(v, s + kPart, 64), v2 = __shfl(v, s + 2 * kPart, 64);
  return (v + v1) + v2;
}

// (theta - T) z = y for symmetric tridiagonal T (diagonal d, off-diagonal e) by
// one wave: a twisted factorisation without pivoting, lanes below 32 from the
// first row and the others from the last, meeting in row n / 2 - which halves
// the chain of dependent divides.  Pivots are kept at |p| >= floor (1e-8 for
// the correction, like the diagonal one; a tiny relative floor for inverse
// iteration).  In the Davidson iteration theta never exceeds the lowest
// eigenvalue of T, so theta - T is negative semidefinite and the sweep is
// stable.
__device__ inline double floored(double p, double floor) {
  return fabs(p) < floor ? (p < 0 ? -floor : floor) : p;
}
// 1/x to about one unit in the last place: the hardware's estimate and two
// Newton steps (a third of the latency of a divide).  It enters reflectors,
// guesses and corrections only; energies and vectors are Rayleigh-Ritz pairs of
// the sigma vectors.
__device__ inline double newton_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
// LDS written by one lane of a wave and read by another
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
struct TwistedTri {      // of one lane
  int n, steps;          // rows, rows of this half
  double l0, l1;         // multipliers of the middle row with either half
};
// ll, ip, bb (LDS, n each): multiplier with the row before, 1/pivot and
// off-diagonal over pivot.  n >= 2; all 64 lanes.
__device__ inline TwistedTri twisted_factor(const double* d, const double* e, int n, double theta,
                                            double floor, double* ll, double* ip, double* bb) {
  const int back = (threadIdx.x >> 5) & 1, mid = n / 2;
  TwistedTri T;
  T.n = n;
  T.steps = back ? n - 1 - mid : mid;
  double l = 0.0, em = 0.0;
  for (int s = 0; s < mid; ++s) {
    // (past its last row the back half works on a row of the front half, unused)
    const int i = back ? n - 1 - s : s;
    const double p = floored((theta - d[i]) + l * em, floor);
    const double y = newton_rcp(p), en = e[back ? max(i - 1, 0) : i];
    if (s < T.steps) {
      ll[i] = l;
      ip[i] = y;
      bb[i] = en * y;
      em = en;
      l = -en * y;
    }
  }
  const double c = l * em;
  T.l0 = lane_value(l, 0);
  T.l1 = lane_value(l, 32);
  const double p = floored((theta - d[mid]) + (lane_value(c, 0) + lane_value(c, 32)), floor);
  ip[mid] = newton_rcp(p);
  wave_lds_fence();
  return T;
}
// z (LDS) on entry y, on return the solution.
__device__ inline void twisted_solve(const TwistedTri& T, const double* ll, const double* ip,
                                     const double* bb, double* z) {
  const int back = (threadIdx.x >> 5) & 1, n = T.n, mid = n / 2;
  const int i0 = back ? n - 1 : 0, di = back ? -1 : 1;
  double v = 0.0;
#pragma unroll 4
  for (int s = 0; s < T.steps; ++s) {
    const int i = i0 + di * s;
    v = z[i] - ll[i] * v;
    z[i] = v;
  }
  v = ((z[mid] - T.l0 * lane_value(v, 0)) - T.l1 * lane_value(v, 32)) * ip[mid];
  z[mid] = v;
#pragma unroll 4
  for (int s = T.steps - 1; s >= 0; --s) {
    const int i = i0 + di * s;
    v = z[i] * ip[i] + bb[i] * v;
    z[i] = v;
  }
  wave_lds_fence();
}

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, class F>
__device__ inline void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}
// Minimum over the 16 lanes of a row, in every lane of it.
__device__ inline double row_min(double x) {
  x = fmin(x, dpp_move<0xB1>(x));
  x = fmin(x, dpp_move<0x4E>(x));
  x = fmin(x, dpp_move<0x141>(x));
  return fmin(x, dpp_move<0x140>(x));
}

// Symmetric Jacobi eigen-solve of the m x m subspace matrix by one wave of
// 64 lanes, parallel ordering: every round applies m/2 disjoint plane
// rotations at once (round-robin pairing of the indices), m-1 rounds per
// sweep.  A rotation is skipped when |a_pq| <= 1e-18 (|a_pp| + |a_qq|) and a
// round without rotations costs only its test; the sweeps stop when a whole
// sweep rotates nothing.  Returns the lowest eigenvalue and its eigenvector
// (ties: lowest index).  Bound by the latency of a round's divides and square
// roots (about 25 rounds at m = 5).
__device__ void wave_jacobi_lowest(double* A, double* B, double* Vm, double* Vt, int m,
                                   double* theta, double* y) {
  const int lane = threadIdx.x & 63;
  __shared__ double rc[kMaxSpace], rt[kMaxSpace];
  __shared__ int partner[kMaxSpace];
  const int N = m + (m & 1);  // even number of players (index m is a dummy when m is odd)
  constexpr int EPL = kMaxSpace * kMaxSpace / 64;  // elements per lane
  int row[EPL], column[EPL];
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    const int e = lane + 64 * u;
    row[u] = e / m;
    column[u] = e % m;
    if (e < m * m) Vm[e] = row[u] == column[u] ? 1.0 : 0.0;
  }
  wave_lds_fence();
  auto wrap = [&](int x) { return x >= N - 1 ? x - (N - 1) : x; };
  for (int sweep = 0; sweep < 40 && N > 1; ++sweep) {
    bool rotated = false;  // uniform
    for (int r = 0; r < N - 1; ++r) {
      // round-robin pairs: position 0 holds index 0, positions 1..N-1 rotate
      const int k = lane < N / 2 ? lane : 0;
      const int a0 = k == 0 ? 0 : 1 + wrap(k - 1 + r), b0 = 1 + wrap(N - 2 - k + r);
      const int p = a0 < b0 ? a0 : b0, q = a0 < b0 ? b0 : a0;
      double apq = 0.0, app = 0.0, aqq = 0.0;
      if (q < m) {
        apq = A[p * m + q];
        app = A[p * m + p];
        aqq = A[q * m + q];
      }
      const bool rot = fabs(apq) > 1e-18 * (fabs(app) + fabs(aqq)) && apq != 0.0;
      if (__ballot(rot) == 0) continue;
      rotated = true;
      if (lane < N / 2) {
        double c = 1.0, t = 0.0;
        if (rot) {
          const double th = (aqq - app) / (2.0 * apq);
          const double tt = (th >= 0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
          c = 1.0 / sqrt(tt * tt + 1.0);
          t = tt * c;
        }
        if (p < m) { partner[p] = rot ? q : p; rc[p] = c; rt[p] = rot ? -t : 0.0; }
        if (q < m) { partner[q] = rot ? p : q; rc[q] = c; rt[q] = rot ? t : 0.0; }
      }
      wave_lds_fence();
      // B = A J, V = V J : column j <- c_j col_j + t_j col_partner(j)
#pragma unroll
      for (int u = 0; u < EPL; ++u) {
        const int e = lane + 64 * u, i = row[u], j = column[u];
        if (e < m * m) {
          const int pj = partner[j];
          B[e] = rc[j] * A[e] + rt[j] * A[i * m + pj];
          Vt[e] = rc[j] * Vm[e] + rt[j] * Vm[i * m + pj];
        }
      }
      wave_lds_fence();
      // A = J^T B : row i <- c_i row_i + t_i row_partner(i)
#pragma unroll
      for (int u = 0; u < EPL; ++u) {
        const int e = lane + 64 * u, i = row[u], j = column[u];
        if (e < m * m) {
          const int pi = partner[i];
          A[e] = rc[i] * B[e] + rt[i] * B[pi * m + j];
          Vm[e] = Vt[e];
        }
      }
      wave_lds_fence();
    }
    if (!rotated) break;
  }
  int best = 0;
  for (int k = 1; k < m; ++k)
    if (A[k * m + k] < A[best * m + best]) best = k;
  *theta = A[best * m + best];
  for (int k = lane; k < m; k += 64) y[k] = Vm[k * m + best];
  wave_lds_fence();
}

// Reduce the dots of the newest column into Hs; when the subspace is
// complete (guess phase) or always (iteration phase), Rayleigh-Ritz.
// One 64-thread block per item.
//
// Restart: a full subspace (mmax vectors) is collapsed onto the Ritz vector
// x = V y (and H x = S y) in slot 0 and the previous iteration's Ritz vector,
// made orthogonal to x, in slot 1: z = yp - (y.yp) y in the subspace's
// orthonormal basis, x' = V z / |z| (kept when |z| > kRestartMin).  The
// projected matrix becomes diag(theta, z^T Hs z / |z|^2): y is an
// eigenvector of Hs and z is orthogonal to it.  The state is that of the
// collapsed subspace from here on; the residual, which reads every vector
// anyway, collapses them (kernels of their own cost 10 us per iteration of
// a small batch and a pass over both vectors of a large one).
constexpr double kRestartMin = 1e-8;
__global__ void k_dav_rr(const Item* __restrict__ items, int ibase,
                         const double* __restrict__ part, DavState* st, int slot, int mmax) {
  const Item& I = items[ibase + blockIdx.x];
  DavState& S = st[ibase + blockIdx.x];
  if (!item_active(S, slot)) return;
  const int j = slot >= 0 ? slot : S.m - 1;
  const int m = j + 1;
  const int lane = threadIdx.x;
  // the Ritz coefficients of the subspace before the newest vector
  const double yold = (lane < kMaxSpace && lane < j) ? S.y[lane] : 0.0;
  const double v = wave_parts(part, I);
  if (lane < m) {
    S.Hs[lane * kMaxSpace + j] = v;
    S.Hs[j * kMaxSpace + lane] = v;
  }
  const bool solve = slot < 0 || slot == S.nguess - 1;
  if (!solve) return;
  __shared__ double A[kMaxSpace * kMaxSpace], B[kMaxSpace * kMaxSpace];
  __shared__ double Vm[kMaxSpace * kMaxSpace], Vt[kMaxSpace * kMaxSpace], y[kMaxSpace];
  __shared__ double zs[kMaxSpace];
  // (the newest row and column from here: their stores may still be under way)
  auto hs = [&](int i, int l, double newest) {
    return i < j && l < j ? S.Hs[i * kMaxSpace + l] : newest;
  };
  for (int k0 = 0; k0 < m * m; k0 += 64) {  // every lane: the newest comes from other lanes
    const int k = k0 + lane, i = k / m, l = k % m;
    const double nv = __shfl(v, i == j ? l : i, 64);
    if (k < m * m) A[k] = hs(i, l, nv);
  }
  wave_lds_fence();
  double th;
  wave_jacobi_lowest(A, B, Vm, Vt, m, &th, y);
  const int q = lane & 15;  // a row of 16 lanes holds the subspace
  const double yq = q < m ? y[q] : 0.0, yo = __shfl(yold, q, 64);
  if (m >= mmax) {
    const double cc = row_sum(yq * yo);
    double z = fma(-cc, yq, yo);
    const double nz = sqrt(row_sum(z * z));
    const bool keep = nz > kRestartMin;
    z = keep ? z / nz : 0.0;
    if (lane < kMaxSpace) zs[q] = z;
    wave_lds_fence();
    // (the store of the newest row and column by this wave comes before)
    double hz = 0.0;
    for (int i = 0; i < m; ++i) {
      const double nv = __shfl(v, q == j ? i : q, 64);
      hz += (q < m ? hs(q, i, nv) : 0.0) * zs[i];
    }
    const double h11 = row_sum(z * hz);
    if (lane < kMaxSpace) {
      S.cy[lane] = yq;
      S.cz[lane] = z;
      S.y[lane] = lane == 0 ? 1.0 : 0.0;
    }
    if (lane == 0) {
      S.Hs[0] = th;
      S.Hs[1] = 0.0;
      S.Hs[kMaxSpace] = 0.0;
      S.Hs[kMaxSpace + 1] = h11;
      S.m = keep ? 2 : 1;
    }
  } else {
    if (lane < kMaxSpace) S.y[lane] = yq;
    if (lane == 0 && slot >= 0) S.m = m;  // end of the guess phase
  }
  if (lane == 0) {
    S.restart = m >= mmax ? m : 0;
    S.theta = th;
    if (slot < 0) S.iters += 1;
  }
}

// One element of an item's collapse (k_dav_rr): x and H x into slot 0, x' and
// H x' into slot 1 when the restart keeps it (m == 2).  v0 / v1: their
// vectors, s0: H x.
template <int M>
__device__ inline void collapse_element(double* __restrict__ Vi, double* __restrict__ Si,
                                        int64_t ntot, const DavState& S, double& v0, double& v1,
                                        double& s0) {
  double x = 0.0, sx = 0.0, xp = 0.0, sxp = 0.0;
  const int n = M > 0 ? M : S.restart;
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const double v = Vi[(int64_t)i * ntot], s = Si[(int64_t)i * ntot];
    x += S.cy[i] * v;
    sx += S.cy[i] * s;
    xp += S.cz[i] * v;
    sxp += S.cz[i] * s;
  }
  Vi[0] = x;
  Si[0] = sx;
  if (S.m == 2) {
    Vi[ntot] = xp;
    Si[ntot] = sxp;
  }
  v0 = x;
  v1 = xp;
  s0 = sx;
}
// f(integral_constant) with the restarts' usual subspace sizes unrolled
template <class F>
__device__ inline void with_restart(int n, F&& f) {
  if (n == 5) f(std::integral_constant<int, 5>{});
  else if (n == 8) f(std::integral_constant<int, 8>{});
  else f(std::integral_constant<int, 0>{});
}

// Residual r = S y - theta V y, preconditioned t = r / (theta - H_II) into
// slot m (after the collapse where the item restarts); partial sums of V_i . t (i < m), |r|^2 (index kMaxSpace) and |t|^2
// (index kMaxSpace + 1).
__global__ void __launch_bounds__(256) k_dav_residual(const Item* __restrict__ items,
                                                      const Work* __restrict__ work, double* V,
                                                      double* Sv,
                                                      const double* __restrict__ diag,
                                                      int64_t ntot,
                                                      const DavState* __restrict__ st,
                                                      double* part) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (S.conv || S.olsen) return;
  const int m = S.m;
  const double th = S.theta;
  if (S.restart) {  // the Ritz vector is slot 0 after the collapse
    double acc[kMaxSpace + 2];
#pragma unroll
    for (int i = 0; i <= kMaxSpace + 1; ++i) acc[i] = 0.0;
    const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
    const int64_t e1 = min(e0 + kChunk, I.ndet);
    with_restart(S.restart, [&](auto mc) {
      for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
        const double d = diag[I.off + e];
        double v0, v1, s0;
        collapse_element<decltype(mc)::value>(V + I.off + e, Sv + I.off + e, ntot, S, v0, v1, s0);
        const double r = s0 - th * v0;
        acc[kMaxSpace] += r * r;
        double den = th - d;
        if (fabs(den) < 1e-8) den = den < 0 ? -1e-8 : 1e-8;
        const double tv = r / den;
        V[(int64_t)m * ntot + I.off + e] = tv;
        acc[kMaxSpace + 1] += tv * tv;
        acc[0] += v0 * tv;
        acc[1] += v1 * tv;
      }
    });
    block_reduce_store<kMaxSpace + 2>(acc, m, kMaxSpace, part + (int64_t)wk.begin * kPart);
    return;
  }
  double y[kMaxSpace];
#pragma unroll
  for (int i = 0; i < kMaxSpace; ++i) y[i] = S.y[i];
  double acc[kMaxSpace + 2];
#pragma unroll
  for (int i = 0; i <= kMaxSpace + 1; ++i) acc[i] = 0.0;
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  double* t_out = V + (int64_t)m * ntot + I.off;
  const bool unrolled = with_space(m, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      double r = 0.0;
      double v[M > 0 ? M : 1];
#pragma unroll
      for (int i = 0; i < M; ++i) {
        v[i] = V[(int64_t)i * ntot + I.off + e];
        r += y[i] * (Sv[(int64_t)i * ntot + I.off + e] - th * v[i]);
      }
      acc[kMaxSpace] += r * r;
      double den = th - diag[I.off + e];
      if (fabs(den) < 1e-8) den = den < 0 ? -1e-8 : 1e-8;
      const double tv = r / den;
      t_out[e] = tv;
      acc[kMaxSpace + 1] += tv * tv;
#pragma unroll
      for (int i = 0; i < M; ++i) acc[i] += v[i] * tv;
    }
  });
  if (!unrolled) {
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      double r = 0.0;
      double v[kMaxSpace];
  #pragma unroll
      for (int i = 0; i < kMaxSpace; ++i) {
        v[i] = 0.0;
        if (i < m) {
          v[i] = V[(int64_t)i * ntot + I.off + e];
          r += y[i] * (Sv[(int64_t)i * ntot + I.off + e] - th * v[i]);
        }
      }
      acc[kMaxSpace] += r * r;
      double den = th - diag[I.off + e];
      if (fabs(den) < 1e-8) den = den < 0 ? -1e-8 : 1e-8;
      const double tv = r / den;
      t_out[e] = tv;
      acc[kMaxSpace + 1] += tv * tv;
  #pragma unroll
      for (int i = 0; i < kMaxSpace; ++i)
        if (i < m) acc[i] += v[i] * tv;
    }
  }
  block_reduce_store<kMaxSpace + 2>(acc, m, kMaxSpace, part + (int64_t)wk.begin * kPart);
}

// Olsen-corrected preconditioner.  With x = V y the Ritz vector and
// r = S y - theta x its residual, the correction is
//   t = -(D - theta)^{-1} (r - eps x),  eps = x^T (D-theta)^{-1} r / x^T (D-theta)^{-1} x,
// the choice that makes t orthogonal to x (Olsen, Jorgensen and Simons'
// correction of the diagonal-preconditioned update used in FCI codes).
// Pass 1 stores r and x and reduces |r|^2, x.(D-theta)^{-1} r, x.(D-theta)^{-1} x.
__device__ inline double guarded_den(double d) {
  return fabs(d) < 1e-8 ? (d < 0 ? -1e-8 : 1e-8) : d;
}

__global__ void __launch_bounds__(256) k_dav_residual_olsen(
    const Item* __restrict__ items, const Work* __restrict__ work, double* V, double* Sv,
    const double* __restrict__ diag, int64_t ntot, const DavState* __restrict__ st,
    double* __restrict__ Rb, double* __restrict__ Xb, double* part, int all) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (S.conv || !(all || S.olsen)) return;
  const int m = S.m;
  const double th = S.theta;
  double y[kMaxSpace];
#pragma unroll
  for (int i = 0; i < kMaxSpace; ++i) y[i] = S.y[i];
  double acc[3] = {0.0, 0.0, 0.0};
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
    double x = 0.0, sx = 0.0;
    if (S.restart) {  // uniform
      double v1;
      collapse_element<0>(V + I.off + e, Sv + I.off + e, ntot, S, x, v1, sx);
    } else {
#pragma unroll
      for (int i = 0; i < kMaxSpace; ++i)
        if (i < m) {
          x += y[i] * V[(int64_t)i * ntot + I.off + e];
          sx += y[i] * Sv[(int64_t)i * ntot + I.off + e];
        }
    }
    const double r = sx - th * x;
    const double den = guarded_den(diag[I.off + e] - th);
    Rb[I.off + e] = r;
    Xb[I.off + e] = x;
    acc[0] += r * r;
    acc[1] += x * r / den;
    acc[2] += x * x / den;
  }
  block_reduce_store<3>(acc, 3, 3, part + (int64_t)wk.begin * kPart);
}

__global__ void k_dav_reduce1_olsen(const Item* __restrict__ items,
                                    const double* __restrict__ part, DavState* st, int ibase,
                                    int nitem, double tol, int max_iter, int all) {
  int it = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);  // a wave per item
  if (it >= nitem) return;
  it += ibase;
  const int lane = threadIdx.x & 63;
  const Item& I = items[it];
  DavState& S = st[it];
  if (S.conv || !(all || S.olsen)) return;
  const double v = wave_parts(part, I);
  const double rr = lane_value(v, 0), a = lane_value(v, 1), b = lane_value(v, 2);
  if (lane != 0) return;
  S.rnorm = sqrt(rr);
  S.eps = (b != 0.0) ? a / b : 0.0;
  if (S.rnorm <= tol || S.m >= I.ndet) {
    S.conv = 1;
  } else if (S.iters >= max_iter) {
    S.conv = 1;
    S.status = 1;
  }
}

// t = -(r - eps x) / (D - theta) into slot m; partial dots V_i . t (i < m)
__global__ void __launch_bounds__(256) k_dav_precond_olsen(
    const Item* __restrict__ items, const Work* __restrict__ work, double* V,
    const double* __restrict__ diag, int64_t ntot, const DavState* __restrict__ st,
    const double* __restrict__ Rb, const double* __restrict__ Xb, double* part, int all) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (S.conv || !(all || S.olsen)) return;
  const int m = S.m;
  const double th = S.theta, eps = S.eps;
  double acc[kMaxSpace];
#pragma unroll
  for (int i = 0; i < kMaxSpace; ++i) acc[i] = 0.0;
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  double* t_out = V + (int64_t)m * ntot + I.off;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
    const double den = guarded_den(diag[I.off + e] - th);
    const double tv = -(Rb[I.off + e] - eps * Xb[I.off + e]) / den;
    t_out[e] = tv;
#pragma unroll
    for (int i = 0; i < kMaxSpace; ++i)
      if (i < m) acc[i] += V[(int64_t)i * ntot + I.off + e] * tv;
  }
  block_reduce_store<kMaxSpace>(acc, m, kMaxSpace, part + (int64_t)wk.begin * kPart);
}

// first Gram-Schmidt coefficients from the partial dots
__global__ void k_dav_reduce_coef(const Item* __restrict__ items, const double* __restrict__ part,
                                  DavState* st, int ibase, int nitem, int all) {
  int it = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);  // a wave per item
  if (it >= nitem) return;
  it += ibase;
  const int lane = threadIdx.x & 63;
  const Item& I = items[it];
  DavState& S = st[it];
  if (S.conv || !(all || S.olsen)) return;
  const double v = wave_parts(part, I);
  if (lane < kMaxSpace) S.coef[lane] = lane < S.m ? v : 0.0;
  if (lane == 0) S.onepass = 0;
}

// Convergence test and first Gram-Schmidt coefficients of an item, by one wave:
// v holds in lane i < m the total of V_i . t, in lane kMaxSpace |r|^2 and in
// lane kMaxSpace + 1 |t|^2.  An unconverged item whose residual fell below
// olsen_below takes the Olsen correction from the next iteration on (0: never).
__device__ inline void dav_test(const Item& I, DavState& S, double v, double tol, int max_iter,
                                double olsen_below) {
  const int lane = threadIdx.x & 63, m = S.m;
  const double rr = lane_value(v, kMaxSpace), tt = lane_value(v, kMaxSpace + 1);
  const double cf = lane < m ? v : 0.0;
  // one Gram-Schmidt pass suffices when it keeps at least half of |t|^2
  // (the Daniel-Gragg-Kaufman-Stewart criterion); |t - V c|^2 = |t|^2 - |c|^2
  const double n1 = tt - wave_sum64(cf * cf);
  if (lane < kMaxSpace) S.coef[lane] = cf;
  if (lane != 0) return;
  S.rnorm = sqrt(rr);
  S.onepass = (n1 >= 0.5 * tt && n1 > 1e-28) ? 1 : 0;
  S.tnorm2 = n1;
  if (S.rnorm <= tol || m >= I.ndet) {
    S.conv = 1;
  } else if (S.iters >= max_iter) {
    S.conv = 1;
    S.status = 1;
  } else if (S.rnorm < olsen_below) {
    S.olsen = 1;
  }
}
// (where no item has a P-space)
__global__ void k_dav_reduce1(const Item* __restrict__ items, const double* __restrict__ part,
                              DavState* st, int ibase, int nitem, double tol, int max_iter,
                              double olsen_below) {
  int it = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);  // a wave per item
  if (it >= nitem) return;
  it += ibase;
  const Item& I = items[it];
  DavState& S = st[it];
  if (S.conv || S.olsen) return;
  dav_test(I, S, wave_parts(part, I), tol, max_iter, olsen_below);
}

// t -= sum_i coef_i V_i ; partial sums of V_i . t and |t|^2 (second pass).
// Items whose first pass suffices (onepass) are normalised here instead.
__global__ void __launch_bounds__(256) k_dav_orth(const Item* __restrict__ items,
                                                  const Work* __restrict__ work, double* V,
                                                  int64_t ntot, const DavState* __restrict__ st,
                                                  double* part) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (S.conv) return;
  const int m = S.m;
  double cf[kMaxSpace];
#pragma unroll
  for (int i = 0; i < kMaxSpace; ++i) cf[i] = S.coef[i];
  if (S.onepass) {
    const double inv = 1.0 / sqrt(S.tnorm2);
    const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
    const int64_t e1 = min(e0 + kChunk, I.ndet);
    double* t = V + (int64_t)m * ntot + I.off;
    const bool unrolled = with_space(m, [&](auto mc) {
      constexpr int M = decltype(mc)::value;
      for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
        double tv = t[e];
#pragma unroll
        for (int i = 0; i < M; ++i) tv -= cf[i] * V[(int64_t)i * ntot + I.off + e];
        t[e] = tv * inv;
      }
    });
    if (!unrolled) {
      for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
        double tv = t[e];
  #pragma unroll
        for (int i = 0; i < kMaxSpace; ++i)
          if (i < m) tv -= cf[i] * V[(int64_t)i * ntot + I.off + e];
        t[e] = tv * inv;
      }
    }
    return;
  }
  double acc[kMaxSpace + 1];
#pragma unroll
  for (int i = 0; i <= kMaxSpace; ++i) acc[i] = 0.0;
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  double* t = V + (int64_t)m * ntot + I.off;
  const bool unrolled = with_space(m, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      double v[M > 0 ? M : 1];
      double tv = t[e];
#pragma unroll
      for (int i = 0; i < M; ++i) {
        v[i] = V[(int64_t)i * ntot + I.off + e];
        tv -= cf[i] * v[i];
      }
      t[e] = tv;
#pragma unroll
      for (int i = 0; i < M; ++i) acc[i] += v[i] * tv;
      acc[kMaxSpace] += tv * tv;
    }
  });
  if (!unrolled) {
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      double v[kMaxSpace];
      double tv = t[e];
  #pragma unroll
      for (int i = 0; i < kMaxSpace; ++i) {
        v[i] = 0.0;
        if (i < m) {
          v[i] = V[(int64_t)i * ntot + I.off + e];
          tv -= cf[i] * v[i];
        }
      }
      t[e] = tv;
  #pragma unroll
      for (int i = 0; i < kMaxSpace; ++i)
        if (i < m) acc[i] += v[i] * tv;
      acc[kMaxSpace] += tv * tv;
    }
  }
  block_reduce_store<kMaxSpace + 1>(acc, m, kMaxSpace, part + (int64_t)wk.begin * kPart);
}

// Second Gram-Schmidt coefficients; the subspace grows by the new vector.
__global__ void k_dav_reduce2(const Item* __restrict__ items, const double* __restrict__ part,
                              DavState* st, int ibase, int nitem) {
  int it = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);  // a wave per item
  if (it >= nitem) return;
  it += ibase;
  const int lane = threadIdx.x & 63;
  const Item& I = items[it];
  DavState& S = st[it];
  if (S.conv) return;
  const int m = S.m;
  if (S.onepass) {
    if (lane == 0) S.m = m + 1;
    return;
  }
  const double v = wave_parts(part, I);
  const double cf = lane < m ? v : 0.0;
  const double n2 = lane_value(v, kMaxSpace) - wave_sum64(cf * cf);
  if (lane < kMaxSpace) S.coef[lane] = cf;
  if (lane != 0) return;
  S.tnorm2 = n2;
  if (!(n2 > 1e-28)) {  // the correction lies in the subspace: accept
    S.conv = 1;
    S.status = 2;
  } else {
    S.m = m + 1;
  }
}

// t -= sum_i coef_i V_i, t /= |t|: the new basis vector, in the last slot of
// the grown subspace.
__global__ void __launch_bounds__(256) k_dav_orth2(const Item* __restrict__ items,
                                                   const Work* __restrict__ work, double* V,
                                                   int64_t ntot, const DavState* __restrict__ st) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  if (S.conv || S.onepass) return;
  const int m = S.m - 1;
  double cf[kMaxSpace];
#pragma unroll
  for (int i = 0; i < kMaxSpace; ++i) cf[i] = S.coef[i];
  const double inv = 1.0 / sqrt(S.tnorm2);
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  double* t = V + (int64_t)m * ntot + I.off;
  const bool unrolled = with_space(m, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      double tv = t[e];
#pragma unroll
      for (int i = 0; i < M; ++i) tv -= cf[i] * V[(int64_t)i * ntot + I.off + e];
      t[e] = tv * inv;
    }
  });
  if (!unrolled) {
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      double tv = t[e];
  #pragma unroll
      for (int i = 0; i < kMaxSpace; ++i)
        if (i < m) tv -= cf[i] * V[(int64_t)i * ntot + I.off + e];
      t[e] = tv * inv;
    }
  }
}
// ------------------------------------------------------------- P-space
// Davidson with a P-space: the np = min(kMaxPspace-ish cap, ndet) determinants
// of lowest diagonal energy (ties: lower address) span a block H_PP of H that
// is diagonalised exactly once per CASCI, H_PP = U diag(lambda) U^T.  It
// supplies (i) the guess, the lowest eigenvector of H_PP plus the
// lowest-diagonal unit vector orthogonalised against it (so every spin and
// spatial symmetry sector of the determinant basis stays in the subspace),
// and (ii) the preconditioner: the correction t = (theta - H)^-1 r is
// approximated by (theta - H_PP)^-1 r on the P block and by the diagonal
// (theta - H_II)^-1 r elsewhere.  The converged eigenpair does not depend on
// either choice, only the number of iterations does.

// Orderable 64-bit key of a double (ascending unsigned order = ascending
// value; -0 and +0 share the key of +0).
__device__ inline uint64_t order_key(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x == 0.0 ? 0.0 : x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// The np lowest of n distinct 96-bit keys (key_at(i) -> order_key(H_II) and
// address) by radix select in 8-bit digits (12 histogram passes: 8 over the
// value key from the top, 4 over the address), then every key up to the np-th
// is collected, unordered, into khi/klo (exactly min(np, n) of them).
// 256 threads.
template <class KeyAt>
__device__ void select_lowest(const KeyAt& key_at, int64_t n, int np, uint64_t* khi,
                              uint32_t* klo) {
  const int t = threadIdx.x;
  __shared__ uint32_t hist[256], wtot[4];
  __shared__ uint64_t pre_hi;
  __shared__ uint32_t pre_lo;
  __shared__ int64_t need;
  __shared__ uint32_t ncol;
  __shared__ int done;
  if (t == 0) { pre_hi = 0; pre_lo = 0; need = np; ncol = 0; done = 0; }
  __syncthreads();
  if (np < n) {
    for (int dg = 0; dg < 12; ++dg) {
      hist[t] = 0;
      __syncthreads();
      const uint64_t ph = pre_hi;
      const uint32_t pl = pre_lo;
      for (int64_t K = t; K < n; K += 256) {
        uint64_t kh;
        uint32_t kl;
        key_at(K, kh, kl);
        bool match;
        int b;
        if (dg < 8) {
          const int sh = 56 - 8 * dg;
          match = dg == 0 || (kh >> (sh + 8)) == (ph >> (sh + 8));
          b = (int)((kh >> sh) & 0xFF);
        } else {
          const int sh = 24 - 8 * (dg - 8);
          match = kh == ph && (dg == 8 || (kl >> (sh + 8)) == (pl >> (sh + 8)));
          b = (int)((kl >> sh) & 0xFF);
        }
        if (match) atomicAdd(&hist[b], 1u);
      }
      __syncthreads();
      // the digit whose running count first reaches `need`: thread t holds
      // digit t, a wave scan and the totals of the lower waves
      const int64_t k = need;
      const uint32_t h = hist[t];
      uint32_t incl = h;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o, 64);
        if ((t & 63) >= o) incl += up;
      }
      if ((t & 63) == 63) wtot[t >> 6] = incl;
      __syncthreads();
      for (int w = 0; w < (t >> 6); ++w) incl += wtot[w];
      const int64_t below = (int64_t)incl - h;
      if (below < k && ((int64_t)incl >= k || t == 255)) {
        need = k - below;
        if (dg < 8) pre_hi |= (uint64_t)t << (56 - 8 * dg);
        else pre_lo |= (uint32_t)t << (24 - 8 * (dg - 8));
        if (need == (int64_t)h) {  // every key with this prefix is wanted
          done = 1;
          if (dg < 8) pre_hi |= (dg < 7 ? (1ull << (56 - 8 * dg)) - 1 : 0);
          pre_lo |= dg < 8 ? ~0u : dg < 11 ? (1u << (24 - 8 * (dg - 8))) - 1 : 0;
        }
      }
      __syncthreads();
      if (done) break;  // uniform
    }
  } else if (t == 0) {
    pre_hi = ~0ull;
    pre_lo = ~0u;
  }
  __syncthreads();
  const uint64_t ph = pre_hi;
  const uint32_t pl = pre_lo;
  for (int64_t K = t; K < n; K += 256) {
    uint64_t kh;
    uint32_t kl;
    key_at(K, kh, kl);
    if (kh < ph || (kh == ph && kl <= pl)) {
      const uint32_t slot = atomicAdd(&ncol, 1u);
      if (slot < (uint32_t)kMaxPspace) { khi[slot] = kh; klo[slot] = kl; }
    }
  }
  __syncthreads();
}

// P-space size requested from the selection: every determinant of a small
// CASCI, else pmax (at least the eight lowest, the unit guesses when the
// P-space is not used).
__device__ __forceinline__ int select_count(int64_t nd, int pmax) {
  return nd <= kMaxPspace ? (int)nd : (pmax > 8 ? pmax : 8);
}

// First phase for CASCIs of more than one chunk: one block per chunk of
// select_chunk addresses writes the chunk's np lowest keys to the
// item's candidate slots (chunk c of an item whose slots start at s:
// slot s + c, kMaxPspace keys each; unused keys are the sentinel ~0, which is
// never selected since the item has at least np real keys).  Work: item,
// chunk index, first slot of the item.
__global__ void __launch_bounds__(256) k_pspace_select_chunk(const Item* __restrict__ items,
                                                             const Work* __restrict__ work,
                                                             int ibase, int nitem,
                                                             const double* __restrict__ diag,
                                                             uint64_t* __restrict__ cand_hi,
                                                             uint32_t* __restrict__ cand_lo,
                                                             int pmax) {
  const Work wk = work[blockIdx.x];
  if (wk.item < ibase || wk.item >= ibase + nitem) return;
  const Item& I = items[wk.item];
  const int np = select_count(I.ndet, pmax);
  const int64_t size = select_chunk(I.ndet), lo = (int64_t)wk.begin * size;
  const int64_t hi = min(I.ndet, lo + size);
  const double* __restrict__ d = diag + I.off;
  __shared__ uint64_t khi[kMaxPspace];
  __shared__ uint32_t klo[kMaxPspace];
  auto key_at = [&](int64_t i, uint64_t& kh, uint32_t& kl) {
    kh = order_key(d[lo + i]);
    kl = (uint32_t)(lo + i);
  };
  const int64_t n = hi - lo;
  select_lowest(key_at, n, np, khi, klo);
  const int got = n < np ? (int)n : np;
  const int64_t s = ((int64_t)wk.end + wk.begin) * kMaxPspace;
  for (int j = threadIdx.x; j < kMaxPspace; j += 256) {
    cand_hi[s + j] = j < got ? khi[j] : ~0ull;
    cand_lo[s + j] = j < got ? klo[j] : ~0u;
  }
}

// Selection of the np lowest (diagonal, address) keys of one item, then a rank
// sort of the np survivors; pidx[item][k] receives the addresses in ascending
// key order.  One 256-thread block per item.  An item with candidate slots
// (cand_slot[item] >= 0, filled by k_pspace_select_chunk) selects among them;
// the others read the diagonal directly.
__global__ void __launch_bounds__(256) k_pspace_select(const Item* __restrict__ items, int ibase,
                                                       const double* __restrict__ diag,
                                                       int32_t* __restrict__ pidx, int pmax,
                                                       const int32_t* __restrict__ cand_slot,
                                                       const uint64_t* __restrict__ cand_hi,
                                                       const uint32_t* __restrict__ cand_lo) {
  const int it = ibase + blockIdx.x;
  const Item& I = items[it];
  const int64_t nd = I.ndet;
  const int np = select_count(nd, pmax);
  const int t = threadIdx.x;
  __shared__ uint64_t khi[kMaxPspace];
  __shared__ uint32_t klo[kMaxPspace];
  const int slot = cand_slot ? cand_slot[it] : -1;
  if (slot >= 0) {
    const int64_t size = select_chunk(nd), nchunk = (nd + size - 1) / size;
    const uint64_t* __restrict__ ch = cand_hi + (int64_t)slot * kMaxPspace;
    const uint32_t* __restrict__ cl = cand_lo + (int64_t)slot * kMaxPspace;
    auto key_at = [&](int64_t i, uint64_t& kh, uint32_t& kl) {
      kh = ch[i];
      kl = cl[i];
    };
    select_lowest(key_at, nchunk * kMaxPspace, np, khi, klo);
  } else {
    const double* __restrict__ d = diag + I.off;
    auto key_at = [&](int64_t i, uint64_t& kh, uint32_t& kl) {
      kh = order_key(d[i]);
      kl = (uint32_t)i;
    };
    select_lowest(key_at, nd, np, khi, klo);
  }
  // rank sort (keys are distinct)
  if (t < np) {
    const uint64_t kh = khi[t];
    const uint32_t kl = klo[t];
    int rank = 0;
    for (int j = 0; j < np; ++j)
      rank += (khi[j] < kh || (khi[j] == kh && klo[j] < kl)) ? 1 : 0;
    pidx[(int64_t)it * kMaxPspace + rank] = (int32_t)kl;
  }
}

// P-space reduction, one block per item: H_PP is reduced to tridiagonal form by
// Householder reflections, H_PP = Q T Q^T (T: diagonal d, off-diagonal e; Q
// accumulated explicitly for a P-space of a larger CASCI).  The lowest
// eigenvalue of T comes from multisection (every thread tests one point per
// round), its eigenvector from inverse iteration; the guess is Q z.  A CASCI of
// at most kMaxPspace determinants is always solved from its whole-space block
// (the guess is then the exact ground state, whatever pmax); larger ones use a
// P-space of min(pmax, ndet / kPspaceRatio) determinants, since the reduction
// costs about P^3 against a Davidson iteration's ndet npair^2; below
// kPspaceMinDim (where small P-spaces can also steer the solver to an excited
// root) they start from `nunit` lowest-diagonal unit vectors with the diagonal
// correction.  The dense vector is always added.  Six instantiations run over
// host-built item lists: three sizes, each for a P-space and for a whole
// space.

// Guess of the CASCIs without a P-space, one 256-thread block per item of
// the view (the others return at once): a single determinant is its own
// solution; otherwise unit vectors on the nunit lowest diagonal determinants
// (idx is sorted) and the dense vector without those components in slot
// nunit.
__global__ void __launch_bounds__(256) k_pspace_guess(const Item* __restrict__ items, int ibase,
                                                      const double* __restrict__ diag,
                                                      const int32_t* __restrict__ pidx, double* V,
                                                      int64_t ntot, DavState* st, int pmax,
                                                      int nunit) {
  const int it = ibase + blockIdx.x;
  const Item& I = items[it];
  DavState& S = st[it];
  const int t = threadIdx.x;
  const int64_t nd = I.ndet;
  const int32_t* __restrict__ idx = pidx + (int64_t)it * kMaxPspace;
  if (nd == 1) {  // nothing to solve: the single determinant
    if (t == 0) {
      V[I.off] = 1.0;
      S.m = 1; S.nguess = 1; S.np = 0; S.iters = 0; S.status = 0; S.rnorm = 0.0; S.conv = 1;
      S.onepass = 0;
      S.olsen = 0;
      S.theta = diag[I.off];
    }
    return;
  }
  if (pspace_dim(nd, pmax) != 0) return;
  const int g = nunit;
  const double sc = 1.0 / sqrt((double)(nd - g));
  double* __restrict__ vr = V + (int64_t)g * ntot + I.off;
  for (int64_t K = t; K < nd; K += 256) {
    bool hit = false;
    for (int j = 0; j < g; ++j) hit |= idx[j] == K;
    vr[K] = hit ? 0.0 : hash_sign(K) * sc;
  }
  if (t < g) V[(int64_t)t * ntot + I.off + idx[t]] = 1.0;
  if (t == 0) {
    S.m = 0; S.nguess = g + 1; S.np = 0; S.iters = 0; S.status = 0; S.rnorm = 0.0; S.conv = 0;
    S.onepass = 0;
    S.olsen = 0;
    S.theta = 0.0;
  }
}

// H_PP of the items of plist, lower triangle, into the rows of pQ that Q takes
// later.  Grid (items, blocks of kMatrixElems elements of the largest P-space
// of the class): an element is a chain of loads (strings, orbitals,
// integrals), so it needs many threads; in the reduction's own block it took
// 28 us at n = 76 and 37 us at n = 112.
constexpr int kMatrixElems = 512;
__global__ void __launch_bounds__(256) k_pspace_matrix(
    const Item* __restrict__ items, const int32_t* __restrict__ plist,
    const ItemHam* __restrict__ hams, const double* __restrict__ diag,
    const int32_t* __restrict__ pidx, double* __restrict__ pQ, int pmax) {
  constexpr int PM = kMaxPspace;
  __shared__ uint64_t sa[PM], sb[PM];
  const int it = plist[blockIdx.x];
  const Item& I = items[it];
  const int n = pspace_dim(I.ndet, pmax), t = threadIdx.x;
  const int x0 = blockIdx.y * kMatrixElems, x1 = min(x0 + kMatrixElems, n * (n + 1) / 2);
  if (I.ndet == 1 || x0 >= x1) return;
  const int32_t* __restrict__ idx = pidx + (int64_t)it * PM;
  for (int k = t; k < n; k += 256) {
    uint64_t ma, mb;
    det_strings(I, idx[k], ma, mb);  // an address of this item: 0 <= idx < ndet
    sa[k] = ma;
    sb[k] = mb;
  }
  __syncthreads();
  const ItemHam& H = hams[I.ham];
  double* __restrict__ A = pQ + (int64_t)it * PM * PM;
  for (int x = x0 + t; x < x1; x += 256) {
    int i = (int)((sqrt(8.0 * x + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= x) ++i;
    while (i * (i + 1) / 2 > x) --i;
    const int j = x - i * (i + 1) / 2;
    A[i * PM + j] = (i == j) ? diag[I.off + idx[i]] : sc_offdiag(H, sa[i], sb[i], sa[j], sb[j]);
  }
}

// One block per item of plist (absolute item indices) with a P-space of at
// most 16 NB determinants, its matrix in the item's rows of pQ.  EXACT: the
// P-space is the whole space; the guess is exact and needs no correction, so
// Q and T are not formed or stored: u = Q z comes from the reflectors, kept
// in LDS.
//
// The block is a chain of n steps, so what counts is the latency of a step.
// The whole symmetric matrix and Q sit in registers, dealt cyclically over 16
// rows x 16 columns of threads: thread (r, c) holds rows r + 16 i, columns
// c + 16 j.  A DPP row of 16 lanes then holds complete matrix rows, so the
// products B v and Q v end in DPP sums, and a step has one barrier: B v and
// the next column go round through LDS together, and every thread brings
// that column up to date for itself.  Q takes each reflector in the same step
// (Q <- Q - (Q v) beta v^T).  Done columns drop out 16 at a time (kb
// and the register indices are constants).  A wave per SIMD:
// more waves repeat the step's scalar part and its LDS reads.
// A matrix packed in LDS with Q in global memory, five barriers per step and
// divides on the eigenvalue's chains took 446 us at n = 76 and 956 us at 112;
// this form with the matrix from k_pspace_matrix takes 106 and 195 us, and
// 0.35 ms instead of 0.69 for the 100-determinant CASCIs of an expansion.
template <int NB, bool EXACT>
__global__ void __launch_bounds__(256, EXACT ? 2 : 1) k_pspace_eigen(
    const Item* __restrict__ items, const int32_t* __restrict__ plist,
    const int32_t* __restrict__ pidx, double* __restrict__ pQ, double* __restrict__ pT, double* V,
    int64_t ntot, DavState* st, int pmax) {
  constexpr int PMAX = 16 * NB, NT = 256;
  constexpr int PM = kMaxPspace;  // stride of the per-item arrays in global memory
  static_assert(PMAX <= PM && PMAX <= NT, "a thread per P row");
  __shared__ double refl[EXACT ? PMAX * (PMAX - 1) / 2 : 1], beta[EXACT ? PMAX : 1];
  __shared__ double pv[2][PMAX], xo[2][PMAX], dd[PMAX], ee[PMAX], es[PMAX], zz[PMAX];
  __shared__ double ll[PMAX], ip[PMAX], bb[PMAX];
  __shared__ int first[2][NT / 64];
  const int it = plist[blockIdx.x];
  const Item& I = items[it];
  DavState& S = st[it];
  const int t = threadIdx.x, r = t >> 4, c = t & 15;
  const int64_t nd = I.ndet;
  const int32_t* __restrict__ idx = pidx + (int64_t)it * PM;
  const int n = pspace_dim(nd, pmax);
  // the list holds only this class (checked again: a mismatch would overrun LDS)
  if (nd == 1 || n == 0 || n > PMAX || (nd == n) != EXACT) return;
  double* __restrict__ Q = pQ + (int64_t)it * PM * PM;
  double a[NB][NB], q[NB][NB];  // rows and columns >= n of a are zero
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int row = r + 16 * i, col = c + 16 * j;
      const int hi = max(row, col), lo = min(row, col);
      const double x = Q[min(hi, n - 1) * PM + min(lo, n - 1)];
      a[i][j] = hi < n ? x : 0.0;
      q[i][j] = row == col ? 1.0 : 0.0;
    }
  if (t < PMAX) ee[t] = 0.0;
  // offset of reflector k's row x (x = k + 1 .. PMAX - 1) in refl
  auto refl_at = [](int k) { return k * (2 * PMAX - k - 1) / 2 - (k + 1); };

  // ---- Householder reduction: step k annihilates A[k+2.., k].  vr, vc: the
  // column below its diagonal, then the reflector, zero up to row k.
  if (c == 0) {
#pragma unroll
    for (int i = 0; i < NB; ++i) xo[1][r + 16 * i] = a[i][0];
  }
  __syncthreads();
  double vr[NB], vc[NB], x0 = xo[1][1];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    vr[i] = r + 16 * i > 0 ? xo[1][r + 16 * i] : 0.0;
    vc[i] = c + 16 * i > 0 ? xo[1][c + 16 * i] : 0.0;
  }
  static_for<NB>([&](auto block) {
    constexpr int kb = decltype(block)::value;
    for (int kk = 0; kk < 16; ++kk) {
      const int k = 16 * kb + kk;
      if (k + 2 >= n) break;  // uniform
      constexpr double kTiny = 1e-280;  // |x|^2 of a column that is done
      double sq = 0.0;
#pragma unroll
      for (int j = kb; j < NB; ++j) sq += vc[j] * vc[j];
      const double sig = row_sum(sq);
      const bool some = sig > kTiny;  // uniform
      // |x| = sig / sqrt(sig): the estimate of 1/sqrt and two Newton steps
      const double ss = some ? sig : 1.0;
      double y = __builtin_amdgcn_rsq(ss);
      double g = ss * y, h = 0.5 * y;
      double e1 = fma(-h, g, 0.5);
      g = fma(g, e1, g);
      h = fma(h, e1, h);
      g = fma(fma(-g, g, ss), h, g);
      const double alpha = x0 >= 0.0 ? -g : g;
      const double bt = some ? newton_rcp(ss - x0 * alpha) : 0.0;
      const double v1 = some ? x0 - alpha : 0.0;
      if (t == 0) ee[k] = some ? alpha : x0;
#pragma unroll
      for (int j = kb; j < NB; ++j)
        if (j <= kb + 1) {
          if (c + 16 * j == k + 1) vc[j] = v1;
          if (r + 16 * j == k + 1) vr[j] = v1;
        }
      if constexpr (EXACT) {
        const int o = refl_at(k);
        if (r == 0) {
#pragma unroll
          for (int j = kb; j < NB; ++j)
            if (c + 16 * j > k) refl[o + c + 16 * j] = vc[j];
        }
        if (t == 0) beta[k] = bt;
      }
      // p = beta B v and beta Q v
      double pr[NB], qr[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int j = kb; j < NB; ++j) {
          if (i >= kb) s0 += a[i][j] * vc[j];
          if (!EXACT) s1 += q[i][j] * vc[j];
        }
        pr[i] = i >= kb ? bt * row_sum(s0) : 0.0;
        qr[i] = !EXACT ? bt * row_sum(s1) : 0.0;
      }
      // p and column k + 1 as it was before this step
      double* __restrict__ pb = pv[kk & 1];
      double* __restrict__ xb = xo[kk & 1];
      if (c == 0) {
#pragma unroll
        for (int i = kb; i < NB; ++i) pb[r + 16 * i] = pr[i];
      }
      if (c == ((kk + 1) & 15)) {
#pragma unroll
        for (int i = kb; i < NB; ++i)
          xb[r + 16 * i] = kk == 15 && kb + 1 < NB ? a[i][kb + 1 < NB ? kb + 1 : kb] : a[i][kb];
      }
      __syncthreads();
      double wc[NB], xc[NB], xr[NB], kv = 0.0;
#pragma unroll
      for (int j = kb; j < NB; ++j) {
        wc[j] = pb[c + 16 * j];
        xc[j] = xb[c + 16 * j];
        xr[j] = xb[r + 16 * j];
        kv += wc[j] * vc[j];
      }
      const double p1 = pb[k + 1];
      // B -= v w^T + w v^T with w = p - K v (rows up to k of v are zero, so w
      // there does no harm)
      const double Kc = 0.5 * bt * row_sum(kv);
      const double w1 = fma(-Kc, v1, p1);
      double wr[NB], nr[NB], nc[NB];
#pragma unroll
      for (int j = kb; j < NB; ++j) {
        // explicit operations: the row and the column copies of v have to
        // agree to the last bit, a difference would grow by |B| per step
        wc[j] = fma(-Kc, vc[j], wc[j]);
        wr[j] = fma(-Kc, vr[j], pr[j]);
        // column k + 1 after this step
        nc[j] = c + 16 * j > k + 1 ? fma(-vc[j], w1, fma(-wc[j], v1, xc[j])) : 0.0;
        nr[j] = r + 16 * j > k + 1 ? fma(-vr[j], w1, fma(-wr[j], v1, xr[j])) : 0.0;
      }
      const double xs = kk >= 14 && kb + 1 < NB ? nc[kb + 1 < NB ? kb + 1 : kb] : nc[kb];
      x0 = lane_value(xs, (k + 2) & 15);
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = kb; j < NB; ++j) {
          if (i >= kb) a[i][j] -= vr[i] * wc[j] + wr[i] * vc[j];
          if (!EXACT) q[i][j] -= qr[i] * vc[j];
        }
#pragma unroll
      for (int j = kb; j < NB; ++j) {
        vc[j] = nc[j];
        vr[j] = nr[j];
      }
    }
  });
  if (t == 0) ee[n - 2] = x0;
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (r == c) dd[r + 16 * i] = a[i][i];
  __syncthreads();
  // ---- lowest eigenvalue of T: multisection on [lo, hi] (Gershgorin)
  double glo = 1e300, ghi = 1e300, gsc = 0.0;
  for (int i = c; i < n; i += 16) {
    const double el = i > 0 ? fabs(ee[i - 1]) : 0.0, er = fabs(ee[i]);
    glo = fmin(glo, dd[i] - (el + er));
    ghi = fmin(ghi, -(dd[i] + (el + er)));
    gsc = fmin(gsc, -(fabs(dd[i]) + 2.0 * er));
  }
  glo = row_min(glo);  // (DPP: with every lane active); the same in every row
  ghi = -row_min(ghi);
  const double scale = -row_min(gsc);
  if (t < PMAX) {
    es[t] = t > 0 && t < n ? ee[t - 1] * ee[t - 1] : 0.0;
    // rows past n keep the sign of the minor before them
    if (t >= n) dd[t] = ghi + (1.0 + scale);
  }
  __syncthreads();
  // 7 rounds of 256 points narrow the interval by 256^7 >= 1.8e16, to the
  // rounding level of the spectrum
  double lo = glo, hi = ghi;  // the same in every thread
  for (int round = 0; round < 7; ++round) {
    const double x = lo + (hi - lo) * (double)(t + 1) / (double)NT;
    // an eigenvalue at or below x: a leading minor of T - x that is not
    // positive.  The minors' own recurrence has one multiply-add on its chain
    // per row (their ratios have a divide); rescaled every eight rows.
    double pm = 0.0, p = 1.0, mn = 1.0;
    for (int i0 = 0; i0 < n; i0 += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double pn = (dd[i0 + u] - x) * p - es[i0 + u] * pm;
        pm = p;
        p = pn;
        mn = fmin(mn, p);
      }
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pm)));
      p = __builtin_amdgcn_ldexp(p, ex);
      pm = __builtin_amdgcn_ldexp(pm, ex);
    }
    // the lowest point with an eigenvalue at or below it ends the interval, the
    // point before it begins it.  One choice for the block: that the test is
    // monotone in x under rounding is not known, and neighbouring points are
    // an ulp apart in the last round.
    const unsigned long long below = __ballot(!(mn > 0.0));
    int* fw = first[round & 1];
    if ((t & 63) == 0) fw[t >> 6] = below ? t + __builtin_ctzll(below) : NT;
    __syncthreads();
    int f = fw[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) f = min(f, fw[w]);
    if (f < NT) {
      const double l = lo;
      lo = l + (hi - l) * (double)f / (double)NT;
      hi = l + (hi - l) * (double)(f + 1) / (double)NT;
    }
  }
  const double lam0 = 0.5 * (lo + hi);
  // ---- eigenvector of T for lam0 by one wave: inverse iteration,
  // (lam0 - T) z = z, with pivots floored at 1e-15 of the spectrum's scale (at
  // least 1e-115: their reciprocals' squares, summed below, have to be finite
  // where T vanishes)
  if (t < 64) {
    const TwistedTri T =
        twisted_factor(dd, ee, n, lam0, 1e-15 * fmax(scale, 1e-100), ll, ip, bb);
    for (int i = t; i < n; i += 64) zz[i] = 1.0;
    wave_lds_fence();
    for (int rep = 0; rep < 3; ++rep) {
      twisted_solve(T, ll, ip, bb, zz);
      double s2 = 0.0;
      for (int i = t; i < n; i += 64) s2 += zz[i] * zz[i];
      const double inv = 1.0 / sqrt(wave_sum64(s2));
      for (int i = t; i < n; i += 64) zz[i] *= inv;
      wave_lds_fence();
    }
    if constexpr (EXACT) {
      // u = H_0 (H_1 (... (H_{n-3} z))), H_k = I - beta_k v_k v_k^T
      static_assert(!EXACT || PMAX <= 128, "two rows per lane");
      double u0 = t < n ? zz[t] : 0.0, u1 = t + 64 < n ? zz[t + 64] : 0.0;
      auto v_at = [&](int k, int row) {
        return row > k && row < n ? refl[refl_at(k) + row] : 0.0;
      };
      double a0 = 0.0, a1 = 0.0;
      if (n > 2) {
        a0 = v_at(n - 3, t);
        a1 = v_at(n - 3, t + 64);
      }
      for (int k = n - 3; k >= 0; --k) {
        const double b0 = a0, b1 = a1, bt = beta[k];
        if (k > 0) {
          a0 = v_at(k - 1, t);
          a1 = v_at(k - 1, t + 64);
        }
        const double sc = bt * wave_sum64(b0 * u0 + b1 * u1);
        u0 -= sc * b0;
        u1 -= sc * b1;
      }
      if (t < n) pv[0][t] = u0;
      if (t + 64 < n) pv[0][t + 64] = u1;
    }
  }
  __syncthreads();
  // ---- outputs: T, Q and the guess vectors
  if constexpr (!EXACT) {
    double* __restrict__ To = pT + (int64_t)it * 2 * PM;
    if (t < n) {
      To[t] = dd[t];
      To[PM + t] = ee[t];
    }
    // u = Q z (row k: P position k)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      double u = 0.0;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int row = r + 16 * i, col = c + 16 * j;
        u += col < n ? q[i][j] * zz[col] : 0.0;
        if (row < n && col < n) Q[row * PM + col] = q[i][j];
      }
      u = row_sum(u);
      if (c == 0) pv[0][r + 16 * i] = u;
    }
    __syncthreads();
  }
  // guess 0: the P-space eigenvector u; guess 1: the dense vector
  // r = sign/sqrt(ndet) minus its component on u (u lives on the P block),
  // |r - c u|^2 = 1 - c^2
  const double* __restrict__ u = pv[0];
  double* __restrict__ v0 = V + I.off;
  if (t < n) v0[idx[t]] = u[t];
  const double rs = 1.0 / sqrt((double)nd);
  double c0 = 0.0;
  for (int k = c; k < n; k += 16) c0 += u[k] * hash_sign(idx[k]) * rs;
  c0 = row_sum(c0);
  const double rest = 1.0 - c0 * c0;
  const bool dense = nd > n && rest > 1e-6;
  if (dense) {
    const double rn = 1.0 / sqrt(rest);
    double* __restrict__ v1 = V + ntot + I.off;
    for (int64_t K = t; K < nd; K += NT) v1[K] = hash_sign(K) * rs * rn;
    __syncthreads();   // the P-block entries below overwrite the dense pass
    if (t < n) v1[idx[t]] = (hash_sign(idx[t]) * rs - c0 * u[t]) * rn;
  }
  if (t == 0) {
    S.m = 0;
    S.nguess = 1 + (dense ? 1 : 0);
    S.np = EXACT ? 0 : n;  // an exact guess needs no P-space correction
    S.onepass = 0;
    S.olsen = 0;
    S.iters = 0;
    S.status = 0;
    S.rnorm = 0.0;
    S.conv = 0;
    S.theta = 0.0;
  }
}

// P-space correction and first Gram-Schmidt coefficients, run after
// k_dav_residual: one block per item with a P-space (the lists of ps), then
// blocks of one wave per item for the others.  On the P block the diagonal correction
// is replaced by t_P = Q (theta - T)^-1 Q^T r_P = (theta - H_PP)^-1 r_P, and the
// change of the dots V_i . t (i < m) and of |t|^2 enters the item's totals.
//
// A chain of short steps, so what counts is that each has its loads in flight
// at once: waves 0..3 hold Q in registers (16 x 16 threads, dealt cyclically)
// from one pass over it and use it for both products, wave 4 sums the chunk
// partials and factors theta - T meanwhile.  (A thread per row or column
// walking Q twice and a serial solve: 18.5 us at n = 76, 28 us at n = 112, and
// 4.6 us of a reduction after it; now 12.5 and 18.2 us.)
template <int NB>
__device__ inline void pspace_products(const double* __restrict__ Qi, int np, double (&q)[NB][NB]) {
  const int r = (threadIdx.x >> 4) & 15, c = threadIdx.x & 15;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int row = r + 16 * i, col = c + 16 * j;
      const double x = Qi[min(row, np - 1) * kMaxPspace + min(col, np - 1)];
      q[i][j] = row < np && col < np ? x : 0.0;
    }
}
constexpr int kCorrectThreads = 320;
__global__ void __launch_bounds__(kCorrectThreads) k_pspace_correct(
    const Item* __restrict__ items, int ibase, int nitem, PspaceArgs ps, double* V,
    const double* __restrict__ Sv, int64_t ntot, const double* __restrict__ part, DavState* st,
    double tol, int max_iter, double olsen_below) {
  constexpr int PM = kMaxPspace;
  __shared__ double rr[PM], zz[PM], tn[PM], zp[16][PM], dd[PM], ee[PM], ll[PM], ip[PM], bb[PM];
  __shared__ double dots[2][kMaxSpace + 1];
  const int32_t* __restrict__ pidx = ps.pidx;
  const double* __restrict__ pT = ps.pT;
  const int t = threadIdx.x, listed = ps.n[0] + ps.n[1] + ps.n[2];
  int b = blockIdx.x;
  if (b >= listed) {  // items without a P-space, one per wave
    const int j = (b - listed) * (kCorrectThreads / 64) + (t >> 6);
    if (j >= nitem) return;
    const int i = ibase + j;
    DavState& S = st[i];
    if (S.conv || S.olsen || S.np > 0) return;
    dav_test(items[i], S, wave_parts(part, items[i]), tol, max_iter, olsen_below);
    return;
  }
  int q = 0;
  while (b >= ps.n[q]) b -= ps.n[q++];
  const int it = ps.list[q][b];
  const Item& I = items[it];
  DavState& S = st[it];
  if (S.conv || S.olsen || S.np == 0) return;
  const int np = S.np, m = S.m;
  const double th = S.theta;
  double total = 0.0;
  TwistedTri T{};
  if (t >= 256) {
    const int lane = t & 63;
    for (int i = lane; i < np; i += 64) {
      dd[i] = pT[(int64_t)it * 2 * PM + i];
      ee[i] = pT[(int64_t)it * 2 * PM + PM + i];
    }
    wave_lds_fence();
    T = twisted_factor(dd, ee, np, th, 1e-8, ll, ip, bb);
    total = wave_parts(part, I);
  }
  // residual on the P block (a thread per position; the other threads repeat
  // the last one)
  int e = 0;
  double told = 0.0;
  if (t < 128) {
    const int k = min(t, np - 1);
    e = pidx[(int64_t)it * PM + k];
    told = V[(int64_t)m * ntot + I.off + e];
    double rv = 0.0;
    const bool unrolled = with_space(m, [&](auto mc) {
      constexpr int M = decltype(mc)::value;
#pragma unroll
      for (int i = 0; i < M; ++i)
        rv += S.y[i] *
              (Sv[(int64_t)i * ntot + I.off + e] - th * V[(int64_t)i * ntot + I.off + e]);
    });
    if (!unrolled)
      for (int i = 0; i < m; ++i)
        rv += S.y[i] *
              (Sv[(int64_t)i * ntot + I.off + e] - th * V[(int64_t)i * ntot + I.off + e]);
    if (t < PM) rr[t] = t < np ? rv : 0.0;
  }
  // z = Q^T r, (theta - T)^-1 z, t = Q z
  auto products = [&](auto nb) {
    constexpr int NB = decltype(nb)::value;
    const int r = (t >> 4) & 15, c = t & 15;
    double q[NB][NB];
    if (t < 256) pspace_products<NB>(ps.pQ + (int64_t)it * PM * PM, np, q);
    __syncthreads();
    if (t < 256) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < NB; ++i) s += q[i][j] * rr[r + 16 * i];
        zp[r][c + 16 * j] = s;
      }
    }
    __syncthreads();
    if (t < np) {
      double s = 0.0;
#pragma unroll
      for (int u = 0; u < 16; ++u) s += zp[u][t];
      zz[t] = s;
    } else if (t < PM) {
      zz[t] = 0.0;
    }
    __syncthreads();
    if (t >= 256) twisted_solve(T, ll, ip, bb, zz);
    __syncthreads();
    if (t < 256) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) s += q[i][j] * zz[c + 16 * j];
        s = row_sum(s);
        if (c == 0) tn[r + 16 * i] = s;
      }
    }
    __syncthreads();
  };
  if (np <= kPspaceSmall) products(std::integral_constant<int, kPspaceSmall / 16>());
  else if (np <= kPspaceMid) products(std::integral_constant<int, kPspaceMid / 16>());
  else products(std::integral_constant<int, PM / 16>());
  if (t < 128) {
    const bool in = t < np;
    const double tnew = in ? tn[t] : 0.0;
    const double dl = in ? tnew - told : 0.0;
    if (in) V[(int64_t)m * ntot + I.off + e] = tnew;
    const double n2 = wave_sum64(in ? tnew * tnew - told * told : 0.0);
    double* __restrict__ dw = dots[t >> 6];
    if ((t & 63) == 0) dw[kMaxSpace] = n2;
    const bool unrolled = with_space(m, [&](auto mc) {
      constexpr int M = decltype(mc)::value;
      double x[M > 0 ? M : 1];
#pragma unroll
      for (int i = 0; i < M; ++i) x[i] = V[(int64_t)i * ntot + I.off + e] * dl;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const double s = wave_sum64(x[i]);
        if ((t & 63) == 0) dw[i] = s;
      }
    });
    if (!unrolled)
      for (int i = 0; i < m; ++i) {
        const double s = wave_sum64(V[(int64_t)i * ntot + I.off + e] * dl);
        if ((t & 63) == 0) dw[i] = s;
      }
  }
  __syncthreads();
  if (t >= 256) {
    const int lane = t & 63;
    if (lane < m) total += dots[0][lane] + dots[1][lane];
    if (lane == kMaxSpace + 1) total += dots[0][kMaxSpace] + dots[1][kMaxSpace];
    dav_test(I, S, total, tol, max_iter, olsen_below);
  }
}

// ------------------------------------------------------------------- RDMs
// For a converged CASCI vector c (normalised):
//   gamma+_ab  = sum_K c_K D+_ab[K]            (= 2 gamma_ab for a > b, gamma_aa)
//   Gamma+_{ab,cd} = sum_K D+_ab[K] D+_cd[K]   (a symmetric rank-update on FP64 MFMA)
// with gamma_pq = <E_pq>, Gamma_pqrs = <E_pq E_rs> - d_qr gamma_ps.  The CI
// vector itself is carried as row NP of the D+ tile (a padding row), so
// gamma+ is column NP of Gamma+ and Gamma+_{NP,NP} = |c|^2.  Each workgroup
// accumulates the upper 16x16 blocks over its tiles in registers and writes
// one partial; k_rdm_reduce sums the partials in a fixed order.
//
// Bound by the build's loads and the LDS reads of the products, so the size of
// a workgroup is that which gives a SIMD four waves to alternate between: from
// 13 orbitals its LDS leaves one per CU, below two or three.  The next tile's
// entries, c values and c row load under this tile's products.  Measured:
// CAS(14,14) 14.2 ms with 256 threads and every load waited for in the build,
// 5.98 with 512, 4.94 with 1024; Hubbard-16 (10 orbitals) 1.83 ms, 1.56 with
// 256, 1.40 with 512; one CAS(8,8) 57, 44 and 33 us.
constexpr int rdm_threads(int nact) { return nact >= 13 ? 1024 : nact >= 8 ? 512 : 256; }
template <int NACT, int TN, int NT = rdm_threads(NACT)>
__global__ void __launch_bounds__(NT) k_rdm_syrk(const Item* __restrict__ items,
                                                 const Work* __restrict__ work,
                                                 const double* __restrict__ civ,
                                                 double* __restrict__ part) {
  constexpr int NP = NACT * (NACT + 1) / 2;
  constexpr int KPAD = (NP + 15) / 16 * 16;
  constexpr int NRB = KPAD / 16;
  constexpr int NBLK = NRB * (NRB + 1) / 2;   // upper 16x16 blocks
  constexpr int NW = NT / 64;
  constexpr int BPW = (NBLK + NW - 1) / NW;   // blocks per wave
  constexpr int NSUB = NT / TN;
  constexpr int NPER = (NP + NSUB - 1) / NSUB;
  constexpr int LDT = TN + 1;
  constexpr int CMAX = (int)binom_c(NACT, NACT / 2);
  constexpr int CPT = (CMAX + NT - 1) / NT;
  static_assert(NP < KPAD, "the c row needs a padding row");
  static_assert(TN == 64, "a wave per D+ row");
  __shared__ double Ds[KPAD * LDT];
  __shared__ int32_t Tb[NP * TN];
  __shared__ double Cr[CMAX];

  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const double* __restrict__ c = civ + I.off;
  const int Na = I.Na, Nb = I.Nb;
  const int32_t* __restrict__ pA = I.pairA;
  const int32_t* __restrict__ pB = I.pairB;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int col = t % TN;
  const int sub = __builtin_amdgcn_readfirstlane(t / TN);
  const int blk = wk.begin / Na;
  const int Kb0 = blk * TN;
  const int Kb = Kb0 + col;
  const double keep = Kb < Nb ? 1.0 : 0.0;
  const int Kbc = Kb < Nb ? Kb : Nb - 1;
  const double* __restrict__ ca = c + Kbc;
  for (int x = t; x < NP * TN; x += NT) {
    const int ab = x / TN, cc = x - ab * TN;
    const int kb = Kb0 + cc < Nb ? Kb0 + cc : Nb - 1;
    Tb[x] = ldg(pB + ab * Nb + kb);
  }
  for (int x = (NP + 1) * LDT + t; x < KPAD * LDT; x += NT) Ds[x] = 0.0;
  // this wave's output blocks (rb <= cb) in a fixed enumeration
  int brb[BPW], bcb[BPW];
  double4_t acc[BPW];
#pragma unroll
  for (int u = 0; u < BPW; ++u) {
    int id = wave + NW * u, rb = 0;
    while (id >= NRB - rb && rb < NRB) { id -= NRB - rb; ++rb; }
    brb[u] = rb;
    bcb[u] = rb + id;
    acc[u] = (double4_t){0.0, 0.0, 0.0, 0.0};
  }
  int32_t ea[NPER];
  double ga[NPER], cr[CPT];
  auto load = [&](int ka) {  // (unconditional loads: a branch would wait for them)
    const int32_t* __restrict__ pa = pA + ka * NP;
#pragma unroll
    for (int i = 0; i < NPER; ++i) ea[i] = ldc(pa + min(sub + NSUB * i, NP - 1));
#pragma unroll
    for (int i = 0; i < NPER; ++i) ga[i] = ldg(ca + (ea[i] ? (ea[i] >> 1) - 1 : 0) * Nb);
#pragma unroll
    for (int j = 0; j < CPT; ++j) cr[j] = ldg(c + ka * Nb + min(t + NT * j, Nb - 1));
  };
  load(wk.begin - blk * Na);
  for (int tile = wk.begin; tile < wk.end; ++tile) {
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (t + NT * j < Nb) Cr[t + NT * j] = cr[j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NPER; ++i) {
      const int ab = sub + NSUB * i;
      if (ab < NP) {
        const int32_t eb = Tb[ab * TN + col];
        const int jb = eb ? (eb >> 1) - 1 : 0;
        const double fa = ea[i] ? ((ea[i] & 1) ? -keep : keep) : 0.0;
        const double fb = eb ? ((eb & 1) ? -keep : keep) : 0.0;
        Ds[ab * LDT + col] = fa * ga[i] + fb * Cr[jb];
      }
    }
    if (sub == 0) Ds[NP * LDT + col] = keep * Cr[Kbc];
    __syncthreads();
    load(min(tile + 1, wk.end - 1) - blk * Na);
#pragma unroll
    for (int u = 0; u < BPW; ++u) {
      if (wave + NW * u >= NBLK) continue;
      const double* ar = Ds + (brb[u] * 16 + (lane & 15)) * LDT + (lane >> 4);
      const double* br = Ds + (bcb[u] * 16 + (lane & 15)) * LDT + (lane >> 4);
#pragma unroll
      for (int k = 0; k < TN; k += 4)
        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[k], br[k], acc[u], 0, 0, 0);
    }
    // no barrier here: the next tile's Cr stores follow this tile's second
    // barrier, its D+ stores the next first one
  }
  double* out = part + (int64_t)blockIdx.x * KPAD * KPAD;
#pragma unroll
  for (int u = 0; u < BPW; ++u) {
    if (wave + NW * u >= NBLK) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = brb[u] * 16 + (lane >> 4) + 4 * v, cc = bcb[u] * 16 + (lane & 15);
      out[r * KPAD + cc] = acc[u][v];
    }
  }
}

// Sum the partials of every item in work order; fill the lower triangle.
// rdmp: [item][KPAD*KPAD] (KPAD of that item).  Grid (items, blocks of 256
// elements of the largest item): a thread sums one element, eight partials in
// flight (one block per item took 7.9 ms for CAS(14,14)'s 512 partials).
__global__ void __launch_bounds__(256) k_rdm_reduce(
    const Item* __restrict__ items, const int32_t* __restrict__ wlo,
    const int32_t* __restrict__ whi, const double* __restrict__ part,
    const int64_t* __restrict__ poff, double* rdmp, const int64_t* __restrict__ roff) {
  const int it = blockIdx.x;
  const Item& I = items[it];
  const int kp = I.kpad;
  const int x = blockIdx.y * 256 + threadIdx.x;
  if (x >= kp * kp) return;
  const int r = x / kp, cc = x % kp;
  double* __restrict__ out = rdmp + roff[it];
  if (r > cc) return;  // the upper triangle holds the data
  double sacc = 0.0;   // a single determinant has none
  if (I.ndet > 1) {
    // an item's partials follow each other, kp * kp apart
    const int w0 = wlo[it], nw = whi[it] - w0;
    const double* __restrict__ p = part + poff[w0] + x;
    const int64_t step = (int64_t)kp * kp;
    int w = 0;
    for (; w + 7 < nw; w += 8) {
      double y[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = ldg(p + (w + q) * step);
#pragma unroll
      for (int q = 0; q < 8; ++q) sacc += y[q];
    }
    for (; w < nw; ++w) sacc += ldg(p + w * step);
  }
  out[x] = sacc;
  out[cc * kp + r] = sacc;
}

// ------------------------------------------------------ gradient assembly
// Weight of f(U) in L = g_0 E_ref + sum_n g_n E^(n): from the closed form
// E^(n) = sum_{|U| <= n} (-1)^{n-|U|} C(M_exp - |U|, n - |U|) f(U), f(()) = E_ref
// (the Moebius solution of the recursion of Eq. 2).
__global__ void k_mbe_weights(const BucketDev* __restrict__ buckets, int nbucket, int nitem,
                              int nexp, int max_order, const double* __restrict__ g, double* w) {
  int it = blockIdx.x * blockDim.x + threadIdx.x;
  if (it >= nitem) return;
  int b = 0;
  while (b + 1 < nbucket && buckets[b + 1].item0 <= it) ++b;
  const int u = buckets[b].order;
  double acc = (u == 0) ? g[0] : 0.0;
  for (int n = (u > 1 ? u : 1); n <= max_order; ++n) {
    const double cb = (double)binom(nexp - u, n - u);
    acc += (((n - u) & 1) ? -cb : cb) * g[n];
  }
  w[it] = acc;
}

// Orbital class of p in CASCI `it`: >= 0 local active index, -1 frozen
// (doubly occupied), -2 deleted.  A single-determinant CASCI has its active
// orbitals either all occupied or all empty and is treated as frozen/deleted.
__device__ inline int orb_class(const int32_t* __restrict__ act, int n, bool single,
                                uint64_t occmask, int p) {
  if (!single)
    for (int t = 0; t < n; ++t)
      if (act[t] == p) return t;
  return (occmask >> p & 1) ? -1 : -2;
}

// gamma_tu of an item from Gamma+ (column NP holds gamma+ = D+ c)
__device__ inline double act_gamma(const double* __restrict__ R, int kp, int np, int t, int u) {
  const double g = R[pair_index(t, u) * kp + np];
  return t == u ? g : 0.5 * g;
}

// 1/4 [G_pqrs + G_qprs + G_pqsr + G_qpsr] of the full-space 2-RDM of one
// CASCI, G = <E_pq E_rs> - d_qr gamma_ps (frozen orbitals doubly occupied).
__device__ double sym_gamma2(int p, int q, int r, int s, int cp, int cq, int cr, int cs,
                             const double* __restrict__ R, int kp, int np) {
  if (cp == -2 || cq == -2 || cr == -2 || cs == -2) return 0.0;
  if (cp >= 0 && cq >= 0 && cr >= 0 && cs >= 0) {
    const double mpq = cp == cq ? 2.0 : 1.0, mrs = cr == cs ? 2.0 : 1.0;
    double v = mpq * mrs * R[pair_index(cp, cq) * kp + pair_index(cr, cs)];
    if (cq == cr) v -= act_gamma(R, kp, np, cp, cs);
    if (cp == cr) v -= act_gamma(R, kp, np, cq, cs);
    if (cq == cs) v -= act_gamma(R, kp, np, cp, cr);
    if (cp == cs) v -= act_gamma(R, kp, np, cq, cr);
    return 0.25 * v;
  }
  // some index frozen: average the raw element over the four index orders
  const int P[4][4] = {{p, q, r, s}, {q, p, r, s}, {p, q, s, r}, {q, p, s, r}};
  const int C[4][4] = {{cp, cq, cr, cs}, {cq, cp, cr, cs}, {cp, cq, cs, cr}, {cq, cp, cs, cr}};
  double acc = 0.0;
  for (int k = 0; k < 4; ++k) {
    const int a = P[k][0], b = P[k][1], c = P[k][2], d = P[k][3];
    const int ca = C[k][0], cb = C[k][1], cc = C[k][2], cd = C[k][3];
    const bool Fa = ca == -1, Fb = cb == -1, Fc = cc == -1, Fd = cd == -1;
    const bool Aa = ca >= 0, Ab = cb >= 0, Ac = cc >= 0, Ad = cd >= 0;
    double v = 0.0;
    if (Fa && Fb && Fc && Fd) {
      if (a == b && c == d) v = (a == c) ? 2.0 : 4.0;
      else if (a == d && b == c) v = -2.0;
    } else if (Fa && Fb && a == b && Ac && Ad) {
      v = 2.0 * act_gamma(R, kp, np, cc, cd);
    } else if (Fc && Fd && c == d && Aa && Ab) {
      v = 2.0 * act_gamma(R, kp, np, ca, cb);
    } else if (Fb && Fc && b == c && Aa && Ad) {
      v = -act_gamma(R, kp, np, ca, cd);
    } else if (Fa && Fd && a == d && Ab && Ac) {
      v = -act_gamma(R, kp, np, cc, cb);
    }
    acc += v;
  }
  return 0.25 * acc;
}

// Orbitals on which a CASCI's full-space RDMs can be non-zero: its active
// orbitals and the occupied orbitals of the reference determinant (frozen
// when not active); every other orbital is deleted.  A single-determinant
// CASCI counts only the occupied ones (its active orbitals are frozen or
// deleted alike).  One thread per item.
__global__ void k_grad_masks(const Item* __restrict__ items, int nitem,
                             const int32_t* __restrict__ act, uint64_t occmask,
                             uint64_t* __restrict__ live) {
  const int it = blockIdx.x * blockDim.x + threadIdx.x;
  if (it >= nitem) return;
  const Item& I = items[it];
  uint64_t m = occmask;
  if (I.ndet > 1)
    for (int t = 0; t < I.n; ++t) m |= (uint64_t)1 << act[it * kMaxActive + t];
  live[it] = m;
}

// Inverted index: list[v * nitem + k], k < count[v], the items whose live
// mask holds orbital v, in ascending order (one wave per orbital compacts
// the items with a ballot, so the order is fixed).
__global__ void __launch_bounds__(64) k_grad_index(const uint64_t* __restrict__ live, int nitem,
                                                   int32_t* __restrict__ list,
                                                   int32_t* __restrict__ count) {
  const int v = blockIdx.x, lane = threadIdx.x;
  int base = 0;
  for (int it0 = 0; it0 < nitem; it0 += 64) {
    const int it = it0 + lane;
    const bool has = it < nitem && ((live[it] >> v) & 1);
    const uint64_t b = __ballot(has);
    if (has) list[(int64_t)v * nitem + base + __popcll(b & ((1ull << lane) - 1))] = it;
    base += __popcll(b);
  }
  if (lane == 0) count[v] = base;
}

// Inverted lists of orbital pairs u < v (pair number v (v - 1) / 2 + u):
// the items whose live mask holds both, in ascending order, stored one after
// another (pair p at poff[p], pcount[p] entries).  An element with two or
// more distinct orbitals draws on the shortest of its pairs' lists when that
// is shorter than its orbitals' lists: the items that hold two given
// expansion orbitals are far fewer than those that hold one.
__host__ __device__ inline int orb_pair_id(int u, int v) { return v * (v - 1) / 2 + u; }

// pcount of pair (blockIdx.x, blockIdx.y) when x < y; one wave per pair.
__global__ void __launch_bounds__(64) k_grad_pair_count(const uint64_t* __restrict__ live,
                                                        int nitem, int32_t* __restrict__ pcount) {
  const int u = blockIdx.x, v = blockIdx.y, lane = threadIdx.x;
  if (u >= v) return;
  const uint64_t m = ((uint64_t)1 << u) | ((uint64_t)1 << v);
  int n = 0;
  for (int it0 = 0; it0 < nitem; it0 += 64) {
    const int it = it0 + lane;
    n += __popcll(__ballot(it < nitem && (live[it] & m) == m));
  }
  if (lane == 0) pcount[orb_pair_id(u, v)] = n;
}

// poff[p] = pcount[0] + ... + pcount[p - 1] for p <= npair: one wave, lane
// l sums a contiguous chunk, the chunk sums are scanned across the lanes.
__global__ void __launch_bounds__(64) k_grad_pair_scan(const int32_t* __restrict__ pcount,
                                                       int npair, int64_t* __restrict__ poff) {
  const int lane = threadIdx.x;
  const int per = (npair + 63) / 64;
  const int lo = min(lane * per, npair), hi = min(lo + per, npair);
  int64_t sum = 0;
  for (int i = lo; i < hi; ++i) sum += pcount[i];
  int64_t incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  int64_t run = incl - sum;
  for (int i = lo; i < hi; ++i) {
    poff[i] = run;
    run += pcount[i];
  }
  if (lane == 63) poff[npair] = incl;
}

// The list of pair (blockIdx.x, blockIdx.y), x < y, compacted with a ballot
// in ascending item order; one wave per pair.
__global__ void __launch_bounds__(64) k_grad_pair_fill(const uint64_t* __restrict__ live,
                                                       int nitem, const int64_t* __restrict__ poff,
                                                       int32_t* __restrict__ plist) {
  const int u = blockIdx.x, v = blockIdx.y, lane = threadIdx.x;
  if (u >= v) return;
  const uint64_t m = ((uint64_t)1 << u) | ((uint64_t)1 << v);
  int32_t* __restrict__ out = plist + poff[orb_pair_id(u, v)];
  int base = 0;
  for (int it0 = 0; it0 < nitem; it0 += 64) {
    const int it = it0 + lane;
    const bool has = it < nitem && (live[it] & m) == m;
    const uint64_t b = __ballot(has);
    if (has) out[base + __popcll(b & ((1ull << lane) - 1))] = it;
    base += __popcll(b);
  }
}

struct GradLists {
  const uint64_t* live;
  const int32_t* list;    // [M][nitem] per-orbital lists
  const int32_t* count;   // [M]
  const int32_t* plist;   // pair lists, concatenated
  const int64_t* poff;    // [npair + 1]
  const int32_t* pcount;  // [npair]
};

// The candidate items of an element with orbitals in mask e: the shortest of
// the inverted lists of its orbitals (ties: the lower orbital) and of its
// orbital pairs (ties: a single orbital, then the earlier pair in
// (lower, higher) order); an item of that list contributes only if its live
// mask holds all of e.  Wave-uniform.
__device__ inline const int32_t* grad_candidates(uint64_t e, int nitem, const GradLists& L,
                                                 int* ncand) {
  int o[4], d = 0;
  for (uint64_t m = e; m; m &= m - 1) o[d++] = __builtin_ctzll(m);
  int best = o[0], nb = L.count[o[0]];
  for (int i = 1; i < d; ++i)
    if (L.count[o[i]] < nb) best = o[i], nb = L.count[o[i]];
  const int32_t* cand = L.list + (int64_t)best * nitem;
  for (int i = 0; i < d; ++i)
    for (int j = i + 1; j < d; ++j) {
      const int pid = orb_pair_id(o[i], o[j]);
      const int np = L.pcount[pid];
      if (np < nb) nb = np, cand = L.plist + L.poff[pid];
    }
  *ncand = nb;
  return cand;
}

// Row and column of entry x of a lower triangle numbered row by row
// (x = i (i + 1) / 2 + j, j <= i).
__device__ inline void tri_index(int64_t x, int* i, int* j) {
  int a = (int)((sqrt(8.0 * (double)x + 1.0) - 1.0) * 0.5);
  while ((int64_t)a * (a + 1) / 2 > x) --a;
  while ((int64_t)(a + 1) * (a + 2) / 2 <= x) ++a;
  *i = a;
  *j = (int)(x - (int64_t)a * (a + 1) / 2);
}

// dE/dh_pq = sum_it w_it gamma_full(p, q), for p >= q, written to (p, q)
// and (q, p).  One block of T threads per element: thread l sums the candidate
// items l, l + T, ... (in ascending item order), then the threads' sums meet in
// block_sum (a fixed order, so the result is bitwise reproducible).  A
// candidate is a chain of loads and there are few elements, so T is large:
// Hubbard-12 (78 elements, 2,510 CASCIs) 98 us with 64, 22 with 512.
constexpr int kGradHThreads = 512;
// Sum over the block, in thread 0.
template <int T>
__device__ inline double block_sum(double v) {
  __shared__ double part[T / 64];
  v = wave_sum64(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = part[0];
#pragma unroll
  for (int i = 1; i < T / 64; ++i) s += part[i];
  return s;
}
__global__ void __launch_bounds__(kGradHThreads) k_grad_h(const Item* __restrict__ items, int nitem,
                                               const int32_t* __restrict__ act, uint64_t occmask,
                                               int M, const double* __restrict__ w,
                                               const double* __restrict__ rdmp,
                                               const int64_t* __restrict__ roff, GradLists L,
                                               double* out) {
  int p, q;
  tri_index(blockIdx.x, &p, &q);
  const int lane = threadIdx.x;
  const uint64_t e = ((uint64_t)1 << p) | ((uint64_t)1 << q);
  int nv;
  const int32_t* __restrict__ cand = grad_candidates(e, nitem, L, &nv);
  double acc = 0.0;
  for (int k = lane; k < nv; k += kGradHThreads) {
    const int it = cand[k];
    if (e & ~L.live[it]) continue;
    const double wt = w[it];
    if (wt == 0.0) continue;
    const Item& I = items[it];
    const bool single = I.ndet == 1;
    const int32_t* a = act + it * kMaxActive;
    const int cp = orb_class(a, I.n, single, occmask, p), cq = orb_class(a, I.n, single, occmask, q);
    double val = 0.0;
    if (cp == -1 && cq == -1 && p == q) val = 2.0;
    else if (cp >= 0 && cq >= 0) val = act_gamma(rdmp + roff[it], I.kpad, I.npair, cp, cq);
    acc += wt * val;
  }
  acc = block_sum<kGradHThreads>(acc);
  if (lane == 0) {
    out[p * M + q] = acc;
    out[q * M + p] = acc;
  }
}

// dE/d(pq|rs) = sum_it w_it 1/2 Sym8(Gamma_full)_pqrs.  The value has the
// 8-fold symmetry of the integrals, so it is formed once per orbit (p >= q,
// r >= s, pair pq >= pair rs) and written to all eight positions; W waves per
// orbit (4 / W orbits per 256-thread block): one where the orbits fill the
// device, four where they don't (Hubbard-12, 3,081 orbits: 249 us with one,
// 140 with four).  An element with an
// orbital outside every CASCI's live set, or with more expansion orbitals
// than any tuple holds, finds an empty or non-matching candidate list.
template <int W>
__global__ void __launch_bounds__(256) k_grad_g(const Item* __restrict__ items, int nitem,
                                                const int32_t* __restrict__ act, uint64_t occmask,
                                                int M, const double* __restrict__ w,
                                                const double* __restrict__ rdmp,
                                                const int64_t* __restrict__ roff, GradLists L,
                                                double* out) {
  const int64_t x = (int64_t)blockIdx.x * (4 / W) + threadIdx.x / (64 * W);
  const int lane = threadIdx.x % (64 * W);
  const int64_t np = (int64_t)M * (M + 1) / 2;
  if (x >= np * (np + 1) / 2) return;  // whole waves; the whole block for W = 4
  int P, Q, p, q, r, s;
  tri_index(x, &P, &Q);
  tri_index(P, &p, &q);
  tri_index(Q, &r, &s);
  const uint64_t e = ((uint64_t)1 << p) | ((uint64_t)1 << q) | ((uint64_t)1 << r) |
                     ((uint64_t)1 << s);
  int nv;
  const int32_t* __restrict__ cand = grad_candidates(e, nitem, L, &nv);
  double acc = 0.0;
  for (int k = lane; k < nv; k += 64 * W) {
    const int it = cand[k];
    if (e & ~L.live[it]) continue;
    const double wt = w[it];
    if (wt == 0.0) continue;
    const Item& I = items[it];
    const bool single = I.ndet == 1;
    const int32_t* a = act + it * kMaxActive;
    const int cp = orb_class(a, I.n, single, occmask, p);
    const int cq = orb_class(a, I.n, single, occmask, q);
    const int cr = orb_class(a, I.n, single, occmask, r);
    const int cs = orb_class(a, I.n, single, occmask, s);
    acc += wt * 0.5 * sym_gamma2(p, q, r, s, cp, cq, cr, cs, rdmp + roff[it], I.kpad, I.npair);
  }
  static_assert(W == 1 || W == 4, "an orbit per wave or per block");
  if constexpr (W == 1) acc = wave_sum64(acc);
  else acc = block_sum<256>(acc);
  if (lane < 8) {
    // lane l writes the permutation (bit 0: swap p q, bit 1: swap r s, bit 2: swap the pairs)
    int a = p, b = q, c = r, d = s;
    if (lane & 1) a = q, b = p;
    if (lane & 2) c = s, d = r;
    if (lane & 4) {
      const int t0 = a, t1 = b;
      a = c, b = d, c = t0, d = t1;
    }
    out[(((int64_t)a * M + b) * M + c) * M + d] = acc;
  }
}

// RDMs of one whole-space CASCI: rdm1 = gamma, rdm2 = Sym8(Gamma).
__global__ void k_casci_rdm_out(const Item* __restrict__ items, int it,
                                const double* __restrict__ rdmp, const int64_t* __restrict__ roff,
                                double* rdm1, double* rdm2) {
  const Item& I = items[it];
  const int n = I.n;
  const double* R = rdmp + roff[it];
  const int64_t n2 = (int64_t)n * n;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n2 * n2;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int p = (int)(x / (n2 * n)), q = (int)((x / n2) % n), r = (int)((x / n) % n),
              s = (int)(x % n);
    if (rdm2) {
      double v;
      if (I.ndet == 1) {
        // every active orbital doubly occupied (nalpha = nbeta = n) or empty
        const bool full = I.na == n;
        v = 0.0;
        if (full) {
          if (p == q && r == s) v = (p == r) ? 2.0 : 4.0;
          else if (p == s && q == r) v = -1.0;  // Sym8 of -2 over the (ij|ji) orbit
          else if ((p == r && q == s) && p != q) v = -1.0;
        }
      } else {
        v = sym_gamma2(p, q, r, s, p, q, r, s, R, I.kpad, I.npair);
      }
      rdm2[x] = v;
    }
    if (rdm1 && x < n2) {
      const int a = (int)(x / n), b = (int)(x % n);
      rdm1[x] = I.ndet == 1 ? ((a == b && I.na == n) ? 2.0 : 0.0)
                            : act_gamma(R, I.kpad, I.npair, a, b);
    }
  }
}

// ---------------------------------------------------------- MBE combine
// f(T) = E_core(T) + theta_T ; eps_T = f(T) - E_ref ;
// Delta eps_T = sum over non-empty U in T of (-1)^{|T|-|U|} eps_U, which is the
// solution of the recursion of Eq. 2 (Moebius inversion of
// eps_T = sum_{non-empty U in T} Delta eps_U).  16 lanes per tuple, subsets dealt
// over them: a thread walking all 2^n of them left the device idle (2,510 tuples
// of order up to 6: 274 -> 34 us).
__global__ void k_item_energy(const Item* __restrict__ items, const ItemHam* __restrict__ hams,
                              const DavState* __restrict__ st, int nitem, double* f) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nitem) return;
  f[i] = hams[items[i].ham].ecore + st[i].theta;
}

__global__ void k_mbe_increments(MbeSpaces sp, const BucketDev* __restrict__ buckets, int nbucket,
                                 const int32_t* __restrict__ tuple_pos, int max_order,
                                 const double* __restrict__ f, int nitem, double* inc,
                                 double* inc_lex, double* f_lex,
                                 const int64_t* __restrict__ order_off,
                                 const int32_t* __restrict__ xpos_o,
                                 const int32_t* __restrict__ xpos_v, int nX) {
  const int it = blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4), lane = threadIdx.x & 15;
  if (it >= nitem || it == 0) return;   // item 0 is the reference CASCI
  const int32_t* tp = tuple_pos + (int64_t)it * (2 * max_order + 2);
  const int no = tp[0], nv = tp[1], n = no + nv;
  const double eref = f[0];
  // bucket base index per (order, nocc)
  double acc = 0.0;
  const unsigned full = (1u << n) - 1u;
  for (unsigned sub = 1 + lane; sub <= full; sub += 16) {
    int co[kMaxActive], cv[kMaxActive];
    int ko = 0, kv = 0;
    for (int b = 0; b < n; ++b)
      if (sub >> b & 1) {
        if (b < no) co[ko++] = tp[2 + b];
        else cv[kv++] = tp[2 + b];
      }
    const int ord = ko + kv;
    int64_t base = -1;
    for (int b = 0; b < nbucket; ++b)
      if (buckets[b].order == ord && buckets[b].nocc == ko) base = buckets[b].item0;
    const int64_t idx = base + comb_lex_rank(co, ko, sp.nXo) * binom(sp.nXv, kv) +
                        comb_lex_rank(cv, kv, sp.nXv);
    const double e = f[idx] - eref;
    acc += ((n - ord) & 1) ? -e : e;
  }
  acc = row_sum(acc);
  if (lane != 0) return;
  inc[it] = acc;
  if (inc_lex) {
    // lexicographic rank of T among the order-n tuples of the sorted X
    int c[kMaxActive];
    for (int b = 0; b < no; ++b) c[b] = xpos_o[tp[2 + b]];
    for (int b = 0; b < nv; ++b) c[no + b] = xpos_v[tp[2 + no + b]];
    for (int a = 1; a < n; ++a) {
      int v = c[a], j = a - 1;
      while (j >= 0 && c[j] > v) { c[j + 1] = c[j]; --j; }
      c[j + 1] = v;
    }
    const int64_t lx = order_off[n - 1] + comb_lex_rank(c, n, nX);
    inc_lex[lx] = acc;
    if (f_lex) f_lex[lx] = f[it];
  }
}

// E^(n) = sum of the order-n increments, one block per order, fixed order.
__global__ void k_mbe_order_sums(const BucketDev* __restrict__ buckets, int nbucket,
                                 const double* __restrict__ inc, double* e_order) {
  const int n = blockIdx.x + 1;
  __shared__ double red[256];
  double acc = 0.0;
  for (int b = 0; b < nbucket; ++b) {
    if (buckets[b].order != n) continue;
    for (int64_t i = threadIdx.x; i < buckets[b].count; i += 256) acc += inc[buckets[b].item0 + i];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) e_order[n - 1] = red[0];
}

// ------------------------------------------------------- bookkeeping kernels
// number of items of [ibase, ibase+nitem) not yet converged (one block)
__global__ void k_count_active(const DavState* __restrict__ st, int ibase, int nitem, int* out) {
  __shared__ int red[256];
  int c = 0;
  for (int i = threadIdx.x; i < nitem; i += 256) c += st[ibase + i].conv ? 0 : 1;
  red[threadIdx.x] = c;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// per-item (iterations, status, guess count, subspace) for the statistics
__global__ void k_collect(const DavState* __restrict__ st, int nitem, int32_t* out) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nitem) return;
  out[4 * i + 0] = st[i].iters;
  out[4 * i + 1] = st[i].status;
  out[4 * i + 2] = st[i].nguess;
  out[4 * i + 3] = st[i].conv;
}

// state of a single caller-provided vector in slot 0 (sigma entry point)
__global__ void k_state_single(DavState* st) {
  if (threadIdx.x == 0) {
    st->m = 1;
    st->nguess = 1;
    st->conv = 0;
    st->iters = 0;
    st->status = 0;
  }
}

// mark every multi-determinant item unconverged (kernel re-timing)
__global__ void k_state_unconv(const Item* __restrict__ items, DavState* st, int nitem) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nitem && items[i].ndet > 1) st[i].conv = 0;
}

// out = s + a*c
__global__ void k_axpy_out(double* out, const double* s, const double* c, double a, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = s[i] + a * c[i];
}

// out = (d + a) * c  (sigma of a diagonal Hamiltonian)
__global__ void k_diag_times(double* out, const double* d, const double* c, double a, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (d[i] + a) * c[i];
}

__global__ void k_add_scalar(double* out, const double* in, double a, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[i] + a;
}

// Ritz vector x = V y of every item into `out` (arena layout), normalised.
__global__ void __launch_bounds__(256) k_ritz_vector(const Item* __restrict__ items,
                                                     const Work* __restrict__ work,
                                                     const double* __restrict__ V, int64_t ntot,
                                                     const DavState* __restrict__ st,
                                                     double* out) {
  const Work wk = work[blockIdx.x];
  const Item& I = items[wk.item];
  const DavState& S = st[wk.item];
  const int64_t e0 = (int64_t)(wk.begin - I.chunk0) * kChunk;
  const int64_t e1 = min(e0 + kChunk, I.ndet);
  for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
    double x = 0.0;
    if (I.ndet == 1) {
      x = 1.0;
    } else {
      for (int i = 0; i < S.m; ++i) x += S.y[i] * V[(int64_t)i * ntot + I.off + e];
    }
    out[I.off + e] = x;
  }
}

// E_total = E_ref + sum_n E^(n), in order
__global__ void k_mbe_total(const double* f, const double* e_order, int k, double* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double e = f[0];
    for (int n = 0; n < k; ++n) e += e_order[n];
    out[0] = f[0];
    out[1] = e;
  }
}

// ------------------------------------------------------- screened expansion
// Set-up from explicit tuples: item i holds the tuple with orbital mask
// masks[i] (bit p = expansion orbital p of the problem; 0 = the reference
// CASCI of R alone).  A = R u T, F = O \ A frozen, the rest deleted.
__global__ void k_mbe_setup_list(MbeSpaces sp, const uint64_t* __restrict__ masks,
                                 const Item* __restrict__ items, const double* __restrict__ h1,
                                 const double* __restrict__ eri, double e_const, ItemHam* hams,
                                 double* warena) {
  const int it = blockIdx.x;
  __shared__ ActiveSet s;
  if (threadIdx.x == 0) {
    const uint64_t m = masks[it];
    uint64_t a = m;
    for (int i = 0; i < sp.nR; ++i) a |= (uint64_t)1 << sp.R[i];
    int nt = 0;
    for (uint64_t x = a; x; x &= x - 1) s.act[nt++] = __builtin_ctzll(x);  // ascending
    s.n = nt;
    s.nf = 0;
    int na = 0;
    for (int i = 0; i < sp.nO; ++i) {
      const int o = sp.O[i];
      if (a >> o & 1) ++na;
      else s.frz[s.nf++] = o;
    }
    s.na = na;
  }
  __syncthreads();
  const Item& I = items[it];
  build_item_hamiltonian(s, sp.M, h1, eri, e_const, I.na + I.nb, &hams[I.ham],
                         pair_matrix(I) ? warena + I.woff : nullptr, I.kpad);
}

// Computed tuples of the lower orders, each order's masks in ascending
// numeric order with their increments.
struct ScreenLevels {
  const uint64_t* mask[kMaxActive + 1];
  const double* inc[kMaxActive + 1];
  int64_t n[kMaxActive + 1];
};

// Eq. 2 over the computed sub-tuples: for tuple i of order k,
// Delta eps = (f_i - E_ref) - sum over its proper non-empty sub-tuples U that
// were computed of Delta eps_U (binary search in U's order; sub-tuples in
// ascending subset order, so the sum has a fixed order).
__global__ void k_screen_increments(const uint64_t* __restrict__ masks, int64_t n, int k,
                                    const double* __restrict__ f, const double* __restrict__ e_ref,
                                    ScreenLevels lv, double* __restrict__ inc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t m = masks[i];
  int bit[kMaxActive];
  int nb = 0;
  for (uint64_t x = m; x; x &= x - 1) bit[nb++] = __builtin_ctzll(x);
  double d = f[i] - e_ref[0];
  const uint32_t full = (1u << k) - 1u;
  for (uint32_t sub = 1; sub < full; ++sub) {
    uint64_t u = 0;
    for (int b = 0; b < k; ++b)
      if (sub >> b & 1) u |= (uint64_t)1 << bit[b];
    const int o = __builtin_popcount(sub);
    const uint64_t* __restrict__ arr = lv.mask[o];
    int64_t lo = 0, hi = lv.n[o];
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (arr[mid] < u) lo = mid + 1;
      else hi = mid;
    }
    if (lo < lv.n[o] && arr[lo] == u) d -= lv.inc[o][lo];
  }
  inc[i] = d;
}

// E^(k) = sum of the order-k increments, in index order (one thread).
// E^(k): one block, every thread a strided partial sum, then a fixed-order
// wave and block reduction (the order depends only on n, so the result is
// reproducible).
__global__ void __launch_bounds__(1024) k_screen_order_sum(const double* __restrict__ inc,
                                                           int64_t n, double* out) {
  __shared__ double part[16];
  const int t = threadIdx.x;
  double e = 0.0;
  for (int64_t i = t; i < n; i += 1024) e += inc[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) e += __shfl_down(e, o, 64);
  if ((t & 63) == 0) part[t >> 6] = e;
  __syncthreads();
  if (t == 0) {
    double sum = 0.0;
    for (int w = 0; w < 16; ++w) sum += part[w];
    out[0] = sum;
  }
}

// ================================================================ launchers
static inline int nblk(int64_t n, int b) { return (int)((n + b - 1) / b); }

void launch_strings(int n, int ne, int64_t N, uint64_t* out, hipStream_t s) {
  if (N > 0) hipLaunchKernelGGL(k_strings, dim3(nblk(N, 256)), dim3(256), 0, s, n, ne, N, out);
}
void launch_links(int n, int ne, int64_t N, uint32_t* packed, uint32_t* packedT, int32_t* abi4,
                  hipStream_t s) {
  if (N > 0)
    hipLaunchKernelGGL(k_links, dim3(nblk(N, 128)), dim3(128), 0, s, n, ne, N, packed, packedT,
                       abi4);
}
void launch_pair_table(int n, int ne, int64_t N, int32_t* out, int32_t* outT, hipStream_t s) {
  if (N > 0)
    hipLaunchKernelGGL(k_pair_table, dim3(nblk(N, 128)), dim3(128), 0, s, n, ne, N, out, outT);
}
void launch_mbe_setup(const MbeSpaces* sp, const BucketDev* buckets, int nbucket, const Item* items,
                      int nitem, const double* h1, const double* eri, double e_const,
                      ItemHam* hams, double* warena, int32_t* tuple_pos, int max_order,
                      int32_t* act_out, hipStream_t s) {
  hipLaunchKernelGGL(k_mbe_setup, dim3(nitem), dim3(256), 0, s, *sp, buckets, nbucket, items, h1,
                     eri, e_const, hams, warena, tuple_pos, max_order, act_out);
}
void launch_casci_setup(int n, const double* const* h1s, const double* const* eris,
                        const double* ecores, const Item* items, int nitem, ItemHam* hams,
                        double* warena, hipStream_t s) {
  hipLaunchKernelGGL(k_casci_setup, dim3(nitem), dim3(256), 0, s, n, h1s, eris, ecores, items,
                     hams, warena);
}
void launch_hdiag(const Item* items, const Work* work, int nwork, const ItemHam* hams,
                  double* diag, hipStream_t s) {
  if (nwork > 0)
    hipLaunchKernelGGL(k_hdiag, dim3(nwork), dim3(256), 0, s, items, work, hams, diag);
}

void launch_string_links(int n, int ne, int64_t N, uint32_t* alpha, uint32_t* beta,
                         hipStream_t s) {
  if (N > 0)
    hipLaunchKernelGGL(k_string_links, dim3(nblk(N, 64)), dim3(64), 0, s, n, ne, N, alpha, beta);
}
void launch_sigma_operands(const Item* items, int nitem, int64_t most, const ItemHam* hams,
                           double* warena, hipStream_t s) {
  // two elements per thread of the largest CASCI
  const int y = (int)(most <= 512 ? 1 : most >= 512 * 256 ? 256 : (most + 511) / 512);
  if (nitem > 0 && most > 0)
    hipLaunchKernelGGL(k_sigma_operands, dim3(nitem, y), dim3(256), 0, s, items, hams, warena);
}
void launch_sigma_same_spin(const Item* items, const Work* work, int nwork, bool small,
                            const double* warena, const double* V, int64_t ntot, double* Sv,
                            const DavState* st, int slot, hipStream_t s) {
  if (nwork <= 0) return;
  if (small)
    hipLaunchKernelGGL((k_sigma_same_spin<1, 1>), dim3(nblk(nwork, 4)), dim3(256), 0, s, items,
                       work, nwork, warena, V, ntot, Sv, st, slot);
  else
    hipLaunchKernelGGL((k_sigma_same_spin<2, 4>), dim3(nblk(nwork, 4)), dim3(256), 0, s, items,
                       work, nwork, warena, V, ntot, Sv, st, slot);
}

template <int NACT, int TN>
static bool sigma_string_t(const Item* items, const Work* work, int nwork, const double* warena,
                           const double* V, int64_t ntot, double* Sv, const DavState* st, int slot,
                           hipStream_t s) {
  if constexpr (TN == 128 && (NACT == 8 || NACT == 9)) {
    return false;  // an option of 128 stands for 64 there (tile_for)
  } else {
    constexpr int WPS = string_wps(NACT, TN), SPW = string_spw(NACT, TN);
    hipLaunchKernelGGL((k_sigma_dgemm<NACT, WPS, SPW>), dim3(nwork), dim3(64 * WPS * SPW), 0, s,
                       items, work, warena, V, ntot, Sv, st, slot);
    return true;
  }
}
template <int NACT>
static bool sigma_string_n(int tn, const Item* items, const Work* work, int nwork,
                           const double* warena, const double* V, int64_t ntot, double* Sv,
                           const DavState* st, int slot, hipStream_t s) {
  switch (tn) {
#define MBEFCI_CASE(T) \
  case T: return sigma_string_t<NACT, T>(items, work, nwork, warena, V, ntot, Sv, st, slot, s);
    MBEFCI_CASE(32) MBEFCI_CASE(64) MBEFCI_CASE(128)
    default: break;
  }
  if constexpr (NACT <= 9) {
    switch (tn) {
      MBEFCI_CASE(-32) MBEFCI_CASE(-64)
      default: break;
    }
  }
#undef MBEFCI_CASE
  return false;
}

template <int NACT, int TN>
static bool sigma_pairs_t(const Item* items, const Work* work, int nwork, const double* warena,
                          const double* V, int64_t ntot, double* G, const DavState* st, int slot,
                          hipStream_t s) {
  if constexpr (TN == 128 && NACT >= 13) {
    return false;  // more LDS than a CU holds
  } else {
    hipLaunchKernelGGL((k_sigma_dgemm_pairrows<NACT, TN>), dim3(nwork), dim3(dgemm_threads(NACT)),
                       0, s, items, work, warena, V, ntot, G, st, slot);
    return true;
  }
}
template <int NACT>
static bool sigma_pairs_n(int tn, const Item* items, const Work* work, int nwork,
                          const double* warena, const double* V, int64_t ntot, double* G,
                          const DavState* st, int slot, hipStream_t s) {
  switch (tn) {
    case 32: return sigma_pairs_t<NACT, 32>(items, work, nwork, warena, V, ntot, G, st, slot, s);
    case 64: return sigma_pairs_t<NACT, 64>(items, work, nwork, warena, V, ntot, G, st, slot, s);
    case 128: return sigma_pairs_t<NACT, 128>(items, work, nwork, warena, V, ntot, G, st, slot, s);
    default: return false;
  }
}

bool launch_sigma_dgemm(int n, int tn, const Item* items, const Work* work, int nwork,
                        const double* warena, const double* V, int64_t ntot, double* G,
                        double* Sv, const DavState* st, int slot, hipStream_t s) {
  if (nwork <= 0) return true;
  switch (n) {
#define MBEFCI_CASE(N) \
  case N: return sigma_string_n<N>(tn, items, work, nwork, warena, V, ntot, Sv, st, slot, s);
    MBEFCI_CASE(2) MBEFCI_CASE(3) MBEFCI_CASE(4) MBEFCI_CASE(5) MBEFCI_CASE(6) MBEFCI_CASE(7)
    MBEFCI_CASE(8) MBEFCI_CASE(9) MBEFCI_CASE(10)
#undef MBEFCI_CASE
#define MBEFCI_CASE(N) \
  case N: return sigma_pairs_n<N>(tn, items, work, nwork, warena, V, ntot, G, st, slot, s);
    MBEFCI_CASE(11) MBEFCI_CASE(12) MBEFCI_CASE(13) MBEFCI_CASE(14)
#undef MBEFCI_CASE
    default: return false;
  }
}

int sym_npc(int npair_class) { return npair_class <= 0 ? 0 : (npair_class + 15) / 16 * 16; }

bool launch_sigma_sym_dgemm(int npc, const Item* items, const Work* work, int nwork,
                            const double* warena, const double* V, int64_t ntot, double* G,
                            const DavState* st, int slot, hipStream_t s) {
  if (nwork <= 0) return true;
  switch (npc) {
#define MBEFCI_CASE(P, T)                                                                     \
  case P:                                                                                     \
    hipLaunchKernelGGL((k_sigma_sym_dgemm<P, T>), dim3(nwork), dim3(256), 0, s, items, work,  \
                       warena, V, ntot, G, st, slot);                                         \
    return true;
    MBEFCI_CASE(16, 64) MBEFCI_CASE(32, 64) MBEFCI_CASE(48, 64) MBEFCI_CASE(64, 32)
    MBEFCI_CASE(80, 32) MBEFCI_CASE(96, 32) MBEFCI_CASE(112, 32)
#undef MBEFCI_CASE
    default: return false;
  }
}

void launch_sigma_sym_gather(const Item* items, const Work* work, int nwork, const double* G,
                             double* Sv, int64_t ntot, const DavState* st, int slot,
                             hipStream_t s) {
  if (nwork > 0)
    hipLaunchKernelGGL(k_sigma_sym_gather, dim3(nwork), dim3(256), 0, s, items, work, G, Sv, ntot,
                       st, slot);
}

void launch_sigma_gather(const Item* items, const Work* work, int nwork, const double* G,
                         double* Sv, int64_t ntot, const DavState* st, int slot, int lds,
                         hipStream_t s) {
  if (nwork > 0)
    hipLaunchKernelGGL(k_sigma_gather, dim3(nwork), dim3(256), lds, s, items, work, G, Sv, ntot,
                       st, slot);
}

// ------------------------------------------------------- peak probes
// Measurement only, off the solver's path.  k_probe_mfma runs independent
// chains of FP64 MFMAs per wave from registers (no memory traffic), of the
// 16x16x4 form or of the 4x4x4 form of four blocks (a quarter of the work each,
// four times as many); the sum is stored only if it equals a value the inputs
// never produce, which keeps the chains live.  k_probe_copy copies 16-byte
// vectors.
constexpr int kProbeMfmaChains = 8;
template <bool BLOCKS4>
__global__ void __launch_bounds__(256) k_probe_mfma(double* out, int iters, double seed) {
  constexpr int CH = kProbeMfmaChains;
  using Acc = std::conditional_t<BLOCKS4, double, double4_t>;
  Acc acc[CH];
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) acc[ch] = Acc{};
  const double a = seed + threadIdx.x * 1e-3, b = 0.5 * seed + threadIdx.x * 1e-4;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int rep = 0; rep < (BLOCKS4 ? 4 : 1); ++rep)
#pragma unroll
      for (int ch = 0; ch < CH; ++ch) {
        if constexpr (BLOCKS4) acc[ch] = mfma4(a, b, acc[ch]);
        else acc[ch] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[ch], 0, 0, 0);
      }
  }
  double s = 0.0;
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    if constexpr (BLOCKS4) s += acc[ch];
    else s += acc[ch][0] + acc[ch][1] + acc[ch][2] + acc[ch][3];
  }
  if (s == -12345.678) out[threadIdx.x] = s;
}
__global__ void __launch_bounds__(256) k_probe_copy(const double2* __restrict__ src,
                                                    double2* __restrict__ dst, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    dst[i] = src[i];
}
void launch_probe_mfma(double* out, int blocks, int iters, bool blocks4, hipStream_t s) {
  if (blocks4)
    hipLaunchKernelGGL(k_probe_mfma<true>, dim3(blocks), dim3(256), 0, s, out, iters, 1.0);
  else
    hipLaunchKernelGGL(k_probe_mfma<false>, dim3(blocks), dim3(256), 0, s, out, iters, 1.0);
}
double probe_mfma_flops(int blocks, int iters) {
  return (double)blocks * 4.0 * iters * kProbeMfmaChains * 2.0 * 16 * 16 * 4;
}
void launch_probe_copy(const double* src, double* dst, int64_t n, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_probe_copy, dim3(blocks), dim3(256), 0, s,
                     reinterpret_cast<const double2*>(src), reinterpret_cast<double2*>(dst), n / 2);
}

void launch_fill(double* p, int64_t n, double v, hipStream_t s) {
  if (n <= 0) return;
  int64_t b = nblk(n, 256);
  if (b > 65536) b = 65536;
  hipLaunchKernelGGL(k_fill, dim3((int)b), dim3(256), 0, s, p, n, v);
}
void launch_dav_guess(const Item* items, int ibase, int nitem, const double* diag, double* V,
                      int64_t ntot, DavState* st, int nguess, hipStream_t s) {
  hipLaunchKernelGGL(k_dav_guess, dim3(nitem), dim3(256), 0, s, items, ibase, diag, V, ntot, st,
                     nguess);
}
void launch_dav_dots(const Item* items, const Work* chunks, int nchunk, const double* V,
                     const double* Sv, int64_t ntot, const DavState* st, int slot, double* part,
                     hipStream_t s) {
  if (nchunk > 0)
    hipLaunchKernelGGL(k_dav_dots, dim3(nchunk), dim3(256), 0, s, items, chunks, V, Sv, ntot, st,
                       slot, part);
}
void launch_dav_rr(const Item* items, int ibase, int nitem, const double* part, DavState* st,
                   int slot, int mmax, hipStream_t s) {
  hipLaunchKernelGGL(k_dav_rr, dim3(nitem), dim3(64), 0, s, items, ibase, part, st, slot, mmax);
}
void launch_pspace_setup(const Item* items, int ibase, int nitem, const PspaceLists& pl,
                         const ItemHam* hams, const double* diag, int32_t* pidx, double* pQ,
                         double* pT, double* V, int64_t ntot, DavState* st, int pmax, int nunit,
                         const PspaceSelect& sel, hipStream_t s) {
  if (sel.nwork > 0)
    hipLaunchKernelGGL(k_pspace_select_chunk, dim3(sel.nwork), dim3(256), 0, s, items, sel.work,
                       ibase, nitem, diag, sel.hi, sel.lo, pmax);
  hipLaunchKernelGGL(k_pspace_select, dim3(nitem), dim3(256), 0, s, items, ibase, diag, pidx, pmax,
                     sel.slot, sel.hi, sel.lo);
  hipLaunchKernelGGL(k_pspace_guess, dim3(nitem), dim3(256), 0, s, items, ibase, diag, pidx, V,
                     ntot, st, pmax, nunit);
  auto reduce = [&](int cls, auto nb, auto exact) {
    constexpr int NB = decltype(nb)::value;
    constexpr int elems = 16 * NB * (16 * NB + 1) / 2;
    if (pl.n[cls] == 0) return;
    hipLaunchKernelGGL(k_pspace_matrix, dim3(pl.n[cls], (elems + kMatrixElems - 1) / kMatrixElems),
                       dim3(256), 0, s, items, pl.list[cls], hams, diag, pidx, pQ, pmax);
    hipLaunchKernelGGL((k_pspace_eigen<NB, decltype(exact)::value>), dim3(pl.n[cls]), dim3(256), 0,
                       s, items, pl.list[cls], pidx, pQ, pT, V, ntot, st, pmax);
  };
  auto size = [&](int cls, auto nb) {
    reduce(2 * cls, nb, std::false_type());
    reduce(2 * cls + 1, nb, std::true_type());
  };
  size(0, std::integral_constant<int, kPspaceSmall / 16>());
  size(1, std::integral_constant<int, kPspaceMid / 16>());
  size(2, std::integral_constant<int, kMaxPspace / 16>());
}
void launch_dav_iteration(const Item* items, int ibase, int nitem, const Work* chunks, int nchunk,
                          double* V, double* Sv, const double* diag, int64_t ntot, DavState* st,
                          double* part, double tol, int max_iter, double* Rb,
                          double* Xb, const PspaceArgs* ps, bool olsen_all, double olsen_below,
                          hipStream_t s) {
  if (nchunk <= 0) return;
  const int nw = nblk(nitem, 4);
  // Olsen-corrected items first (all of them with olsen_all, else those that
  // switched in an earlier iteration), then the diagonal / P-space path for
  // the others, whose test may switch an item for the next iteration
  if (olsen_all || olsen_below > 0.0) {
    const int all = olsen_all ? 1 : 0;
    hipLaunchKernelGGL(k_dav_residual_olsen, dim3(nchunk), dim3(256), 0, s, items, chunks, V, Sv,
                       diag, ntot, st, Rb, Xb, part, all);
    hipLaunchKernelGGL(k_dav_reduce1_olsen, dim3(nw), dim3(256), 0, s, items, part, st, ibase,
                       nitem, tol, max_iter, all);
    hipLaunchKernelGGL(k_dav_precond_olsen, dim3(nchunk), dim3(256), 0, s, items, chunks, V, diag,
                       ntot, st, Rb, Xb, part, all);
    hipLaunchKernelGGL(k_dav_reduce_coef, dim3(nw), dim3(256), 0, s, items, part, st, ibase, nitem,
                       all);
  }
  if (!olsen_all) {
    hipLaunchKernelGGL(k_dav_residual, dim3(nchunk), dim3(256), 0, s, items, chunks, V, Sv, diag,
                       ntot, st, part);
    const int listed = ps ? ps->n[0] + ps->n[1] + ps->n[2] : 0;
    if (listed > 0) {
      const int rest = listed < nitem ? nblk(nitem, kCorrectThreads / 64) : 0;
      hipLaunchKernelGGL(k_pspace_correct, dim3(listed + rest), dim3(kCorrectThreads), 0, s, items,
                         ibase, nitem, *ps, V, Sv, ntot, part, st, tol, max_iter, olsen_below);
    } else
      hipLaunchKernelGGL(k_dav_reduce1, dim3(nw), dim3(256), 0, s, items, part, st, ibase, nitem,
                         tol, max_iter, olsen_below);
  }
  hipLaunchKernelGGL(k_dav_orth, dim3(nchunk), dim3(256), 0, s, items, chunks, V, ntot, st, part);
  hipLaunchKernelGGL(k_dav_reduce2, dim3(nw), dim3(256), 0, s, items, part, st, ibase, nitem);
  hipLaunchKernelGGL(k_dav_orth2, dim3(nchunk), dim3(256), 0, s, items, chunks, V, ntot, st);
}
void launch_item_energy(const Item* items, const ItemHam* hams, const DavState* st, int nitem,
                        double* f, hipStream_t s) {
  hipLaunchKernelGGL(k_item_energy, dim3(nblk(nitem, 64)), dim3(64), 0, s, items, hams, st, nitem,
                     f);
}
void launch_mbe_combine(const MbeSpaces* sp, const BucketDev* buckets, int nbucket,
                        const int32_t* tuple_pos, int max_order, const double* f, int nitem,
                        double* inc, double* inc_lex, double* f_lex, const int64_t* order_off,
                        const int32_t* xpos_o, const int32_t* xpos_v, int nX, double* e_order,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_mbe_increments, dim3(nblk(nitem, 16)), dim3(256), 0, s, *sp, buckets,
                     nbucket, tuple_pos, max_order, f, nitem, inc, inc_lex, f_lex, order_off,
                     xpos_o, xpos_v, nX);
  if (max_order > 0)
    hipLaunchKernelGGL(k_mbe_order_sums, dim3(max_order), dim3(256), 0, s, buckets, nbucket, inc,
                       e_order);
}

}  // namespace mbefci

namespace mbefci {
void launch_count_active(const DavState* st, int ibase, int nitem, int* out, hipStream_t s) {
  hipLaunchKernelGGL(k_count_active, dim3(1), dim3(256), 0, s, st, ibase, nitem, out);
}
void launch_collect(const DavState* st, int nitem, int32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(k_collect, dim3(nblk(nitem, 64)), dim3(64), 0, s, st, nitem, out);
}
void launch_state_single(DavState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_state_single, dim3(1), dim3(64), 0, s, st);
}
void launch_axpy_out(double* out, const double* sv, const double* c, double a, int64_t n,
                     hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_axpy_out, dim3(nblk(n, 256)), dim3(256), 0, s, out, sv, c, a, n);
}
void launch_diag_times(double* out, const double* d, const double* c, double a, int64_t n,
                       hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_diag_times, dim3(nblk(n, 256)), dim3(256), 0, s, out, d, c, a, n);
}
void launch_add_scalar(double* out, const double* in, double a, int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_add_scalar, dim3(nblk(n, 256)), dim3(256), 0, s, out, in, a, n);
}
void launch_ritz_vector(const Item* items, const Work* chunks, int nchunk, const double* V,
                        int64_t ntot, const DavState* st, double* out, hipStream_t s) {
  if (nchunk > 0)
    hipLaunchKernelGGL(k_ritz_vector, dim3(nchunk), dim3(256), 0, s, items, chunks, V, ntot, st,
                       out);
}
void launch_state_unconv(const Item* items, DavState* st, int nitem, hipStream_t s) {
  hipLaunchKernelGGL(k_state_unconv, dim3(nblk(nitem, 64)), dim3(64), 0, s, items, st, nitem);
}
void launch_mbe_total(const double* f, const double* e_order, int k, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_mbe_total, dim3(1), dim3(64), 0, s, f, e_order, k, out);
}
}  // namespace mbefci

namespace mbefci {
template <int NACT, int TN>
static void rdm_syrk_t(const Item* items, const Work* work, int nwork, const double* civ,
                       double* part, hipStream_t s) {
  hipLaunchKernelGGL((k_rdm_syrk<NACT, TN>), dim3(nwork), dim3(rdm_threads(NACT)), 0, s, items,
                     work, civ, part);
}
bool launch_rdm_syrk(int n, int tn, const Item* items, const Work* work, int nwork,
                     const double* civ, double* part, hipStream_t s) {
  if (nwork <= 0) return true;
  if (tn != 64) return false;
  switch (n) {
#define MBEFCI_CASE(N) \
  case N: rdm_syrk_t<N, 64>(items, work, nwork, civ, part, s); return true;
    MBEFCI_CASE(2) MBEFCI_CASE(3) MBEFCI_CASE(4) MBEFCI_CASE(5) MBEFCI_CASE(6) MBEFCI_CASE(7)
    MBEFCI_CASE(8) MBEFCI_CASE(9) MBEFCI_CASE(10) MBEFCI_CASE(11) MBEFCI_CASE(12)
    MBEFCI_CASE(13) MBEFCI_CASE(14)
#undef MBEFCI_CASE
    default: return false;
  }
}
void launch_rdm_reduce(const Item* items, int nitem, const int32_t* wlo, const int32_t* whi,
                       const double* part, const int64_t* poff, double* rdmp, const int64_t* roff,
                       int kpad_max, hipStream_t s) {
  if (nitem > 0)
    hipLaunchKernelGGL(k_rdm_reduce, dim3(nitem, (kpad_max * kpad_max + 255) / 256), dim3(256), 0,
                       s, items, wlo, whi, part, poff, rdmp, roff);
}
void launch_mbe_weights(const BucketDev* buckets, int nbucket, int nitem, int nexp, int max_order,
                        const double* g, double* w, hipStream_t s) {
  hipLaunchKernelGGL(k_mbe_weights, dim3(nblk(nitem, 64)), dim3(64), 0, s, buckets, nbucket, nitem,
                     nexp, max_order, g, w);
}
void launch_grad_index(const Item* items, int nitem, const int32_t* act, uint64_t occmask, int M,
                       uint64_t* live, int32_t* list, int32_t* count, int32_t* pcount,
                       int64_t* poff, hipStream_t s) {
  hipLaunchKernelGGL(k_grad_masks, dim3(nblk(nitem, 64)), dim3(64), 0, s, items, nitem, act,
                     occmask, live);
  hipLaunchKernelGGL(k_grad_index, dim3(M), dim3(64), 0, s, live, nitem, list, count);
  hipLaunchKernelGGL(k_grad_pair_count, dim3(M, M), dim3(64), 0, s, live, nitem, pcount);
  hipLaunchKernelGGL(k_grad_pair_scan, dim3(1), dim3(64), 0, s, pcount, M * (M - 1) / 2, poff);
}
void launch_grad(const Item* items, int nitem, const int32_t* act, uint64_t occmask, int M,
                 const double* w, const double* rdmp, const int64_t* roff, const uint64_t* live,
                 const int32_t* list, const int32_t* count, const int32_t* pcount,
                 const int64_t* poff, int32_t* plist, double* dh, double* dg, hipStream_t s) {
  hipLaunchKernelGGL(k_grad_pair_fill, dim3(M, M), dim3(64), 0, s, live, nitem, poff, plist);
  const GradLists L{live, list, count, plist, poff, pcount};
  const int64_t np = (int64_t)M * (M + 1) / 2;  // p >= q
  hipLaunchKernelGGL(k_grad_h, dim3((int)np), dim3(kGradHThreads), 0, s, items, nitem, act,
                     occmask, M, w, rdmp, roff, L, dh);
  // 8 waves per SIMD x 1024 SIMDs: with fewer orbits a wave each leaves slots.
  // Whole backward with one and four waves: 14 orbitals (5,565 orbits) 330 and
  // 281 us, 16 (9,316) 2.02 and 2.00 ms, 40 (336,610) 0.82 and 1.51 ms.
  const int64_t orbits = np * (np + 1) / 2;
  if (orbits < 8192)
    hipLaunchKernelGGL(k_grad_g<4>, dim3((int)orbits), dim3(256), 0, s, items, nitem, act, occmask,
                       M, w, rdmp, roff, L, dg);
  else
    hipLaunchKernelGGL(k_grad_g<1>, dim3(nblk(orbits, 4)), dim3(256), 0, s, items, nitem, act,
                       occmask, M, w, rdmp, roff, L, dg);
}
void launch_casci_rdm_out(const Item* items, int it, int n, const double* rdmp,
                          const int64_t* roff, double* rdm1, double* rdm2, hipStream_t s) {
  const int64_t n4 = (int64_t)n * n * n * n;
  int b = nblk(n4, 256);
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_casci_rdm_out, dim3(b), dim3(256), 0, s, items, it, rdmp, roff, rdm1, rdm2);
}
void launch_mbe_setup_list(const MbeSpaces* sp, const uint64_t* masks, const Item* items, int nitem,
                           const double* h1, const double* eri, double e_const, ItemHam* hams,
                           double* warena, hipStream_t s) {
  hipLaunchKernelGGL(k_mbe_setup_list, dim3(nitem), dim3(256), 0, s, *sp, masks, items, h1, eri,
                     e_const, hams, warena);
}
void launch_screen_increments(const uint64_t* masks, int64_t n, int k, const double* f,
                              const double* e_ref, const ScreenArrays& lower, double* inc,
                              double* order_sum, hipStream_t s) {
  ScreenLevels lv{};
  for (int o = 0; o <= kMaxActive; ++o) {
    lv.mask[o] = lower.mask[o];
    lv.inc[o] = lower.inc[o];
    lv.n[o] = lower.n[o];
  }
  if (n > 0)
    hipLaunchKernelGGL(k_screen_increments, dim3(nblk(n, 128)), dim3(128), 0, s, masks, n, k, f,
                       e_ref, lv, inc);
  hipLaunchKernelGGL(k_screen_order_sum, dim3(1), dim3(1024), 0, s, inc, n, order_sum);
}
}  // namespace mbefci
