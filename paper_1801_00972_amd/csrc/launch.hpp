// launch.hpp -- host-side entry points of the library's kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "pic_types.hpp"

namespace pic {

// the fixed device scratch array of pic_fields_static (scratch.hip): doubles
// per GPU, 48 MiB; scratch_setup resolves its address on the current device
// (once per device, returns 0 on success), scratch_address returns the kept
// address of a device (nullptr before its set-up)
constexpr size_t kScratchDoubles = size_t(6) << 20;
int scratch_setup(int* device_out, void** addr_out);
void* scratch_address(int device);

// factorisation of the FFT line lengths and lines per block
struct FftPlanHost {
  int nfac_x, fac_x[12];
  int nfac_y, fac_y[12];
  int L_x, L_y;
};

// particles: arrays binned by 4x4x4-cell tile and updated in place (see
// WorkLists); one push block per tile or pair of tiles, the grid padded to a
// multiple of 16
// tiles (plus `extra` padding tiles) rounded up to a multiple of 16
int tile_grid(int nx, int ny, int nz, int extra);
// blocks of the MD kernel; each owns a tally row after the ngrid tile rows
constexpr int kMdTallyRows = 4096;
long sort_keys(int ngrid);                  // ints of sort workspace (tile counts and cursors)
// the streaming kernel (gather, push, walls, candidate test, deposit) of both
// species (descs[0], descs[1] in device memory, L either one's lists); without
// `move` the deposit alone, of the current positions (arrays freshly sorted)
void launch_push(const PushDescF64* descs, const WorkLists& L, bool move, hipStream_t st);
void launch_push(const PushDescF32* descs, const WorkLists& L, bool move, hipStream_t st);
// the push of every (replica, species) of an FP32R ensemble in one launch;
// start[d] is the first work item (push block) of descriptor d, start[ndesc] =
// items the total
void launch_push_batch_f32r(const PushDescF32* descs, const int32_t* start, int ndesc, int items,
                            hipStream_t st);
// the MD particles' sub-cycled motion from P into the other record buffers D
// (beside the push), both species
void launch_md_move(const PartF64 P[2], const PartF64 D[2], const void* E, void* rho,
                    const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                    const WorkLists L[2], hipStream_t st);
void launch_md_move(const PartF32R P[2], const PartF32R D[2], const void* E, void* rho,
                    const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                    const WorkLists L[2], hipStream_t st);
// whether a step's push blocks and MD blocks are few enough for one launch, and
// that launch: launch_push with move and launch_md_move
bool push_md_fits(const MdTables& md, const SpeciesStep& S, const WorkLists& L);
void launch_push_md(const PushDescF64* descs, const PartF64 P[2], const PartF64 D[2], const void* E,
                    void* rho, const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                    const WorkLists L[2], hipStream_t st);
void launch_push_md(const PushDescF32* descs, const PartF32R P[2], const PartF32R D[2],
                    const void* E, void* rho, const MdTables& md, const SpeciesStep S[2],
                    unsigned long long* gc, const WorkLists L[2], hipStream_t st);
// Push and MD motion as two launches side by side: the first enqueued gets the
// chip's waves first.  A long push goes first and hides the MD motion (64x64x256
// cells, 8 grains, FP32R: 1.046 ms a step against 1.119); where the push ends with
// it, the MD kernel's chains go first (36x30x77 cells, 7 per cell, 3 grains, single
// tiles a block: 2.24 ms for 16 steps against 2.27).  The line at 8 million slots
// lies between those two and is no sharp one: boxes of tile pairs with 8 grains take
// less push first on both sides of it (FP32R 2.0, 4.5, 7.6, 15, 32 and 64 million
// slots: 1.6, 1.6, 1.7, 4.4, 10.9 and 6.9 %; FP64 6.9, 2.8, 2.8, 2.4, 2.4, 1.8 %).
// (Two species of up to 2^31 - 1 slots each.)
inline bool push_goes_first(const WorkLists L[2]) {
  return (long)L[0].slots + (long)L[1].slots > 8L << 20;
}
// the push blocks (first tiles) whose window of `margin` cells meets the MD
// cubes' bounding box
std::vector<int32_t> near_blocks(const WorkLists& L, const MdTables& md, int nx, int ny, int nz,
                                 int margin, bool f64);
// whether two window margins give every push block the same window
bool same_windows(const WorkLists& L, int nx, int ny, int nz, int m0, int m1, bool f64);
// everything after the push (descs as in launch_push): the collision candidates
// it had no room for, the outliers, the MD particles' states back from D with
// their collisions, and the next step's MD lists
void launch_lists(const PushDescF64* descs, const PartF64 D[2], bool grains, const WorkLists L[2],
                  int do_mcc, hipStream_t st);
void launch_lists(const PushDescF32* descs, const PartF32R D[2], bool grains, const WorkLists L[2],
                  int do_mcc, hipStream_t st);
// The fields of a step in one launch: phi (the solve's psi lifted with the
// electrode voltages), E = -grad phi into E (FP64 double2 pairs or FP32
// float4), the MD cells' corrected node fields, zero_next (nn 8-byte words,
// may be null) cleared for the next deposit, with it the counts of the lists
// L[].md_next, and, with b, the sums of the
// squared residual b - A psi and of b^2 per block of field_out_sums() blocks.
inline int field_out_planes(int plane, int nz) {
  const long one = (plane + 255) / 256 * (long)(nz + 1);  // blocks of one plane
  return (int)(one < 4096 ? 1 : one >= 16384 ? 8 : one / 2048);
}
inline long field_out_sums(int plane, int nz) {
  const int u = field_out_planes(plane, nz);
  return (plane + 255) / 256 * (long)((nz + u) / u);
}
void launch_field_out(const double* psi, double* phi, void* E, int e_f64,
                      unsigned long long* zero_next, const double* b, double* partials,
                      const MdTables& md, const WorkLists L[2], int nx, int ny, int nz, double dx,
                      RfDrive rf, hipStream_t st);
void launch_init_f64(const PartF64& P, int n, int ppc, int nx, int ny, int sp, uint32_t k0,
                     uint32_t k1, double vth, hipStream_t st);
void launch_init_f32r(const PartF32R& P, int n, int ppc, int nx, int ny, int sp, uint32_t k0,
                      uint32_t k1, double vth, hipStream_t st);
// density and flux moments of one species: mom [4][nn] gets W, v W summed per
// node (added to what it holds, in the rf-phase bin of the step if avg.step
// is set); exactly one of P64, P32 is non-null
int moments_setup();  // the kernels' LDS sizes; 0 or an error
void launch_moments(const PartF64* P64, const PartF32R* P32, const SpeciesStep& S,
                    const WorkLists& L, double* mom, long nn, const AvgBins& avg,
                    hipStream_t st);
// fine-grid moments of both species: mom [2][4][fb.fn] gets W, v W of the
// particles inside the box summed per fine node (added as in launch_moments);
// capacity bounds the slots in use
void launch_fine_moments(const PartF64 P[2], const WorkLists L[2], const FineBox& fb, double* mom,
                         const AvgBins& avg, long capacity, hipStream_t st);
void launch_fine_moments(const PartF32R P[2], const WorkLists L[2], const FineBox& fb, double* mom,
                         const AvgBins& avg, long capacity, hipStream_t st);
// Coulomb collisions (coulomb.hip).  Work buffers of a replica: per species
// the per-cell counts turned into range starts [ncell + 1], fill cursors
// [ncell], each tile's own particles per cell [ncell] (the counting kernel's
// histograms, for the scatter), the (order key, slot) entries [cap] and the
// slots in key order [cap]; the scan's block sums [coulomb_scan_sums(ncell)];
// the pairings performed (accumulated).
struct CoulombBufs {
  int* start[2];
  int* fill[2];
  int* thist[2];
  unsigned long long* key[2];
  int* slot[2];
  int* ord[2];
  int* sums;
  unsigned long long* count;
};
// constants of a pass: pair kinds 0 e-e, 1 Ar+-Ar+, 2 e-Ar+; the variance of
// delta is c_var[kind] n_L / |u|^3 with n_L = (particles) w_vol; species s of
// a pair changes by +- frac[kind][s] du; ncell counts the cells in the tile
// order of the particle bins (64 a tile, the start arrays hold ncell + 1)
struct CoulombConst {
  int ncell;
  uint32_t key0, key1;
  const uint32_t* step;
  double w_vol;
  double c_var[3];
  double frac[3][2];
};
long coulomb_scan_sums(long ncell);
// one pass over both species of a replica; exactly one of P64, P32 is non-null
// (each then points to the two species' arrays); cap bounds the slots in use
void launch_coulomb(const PartF64* P64, const PartF32R* P32, const WorkLists L[2],
                    const CoulombBufs& B, const CoulombConst& C, const long cap[2],
                    hipStream_t st);
// time averages: phi added to its rf-phase bin (avg.stride apart), and one
// sample counted in cnt[bin]
void launch_avg_phi(const double* phi, double* acc, long nn, const AvgBins& avg,
                    unsigned long long* cnt, hipStream_t st);
// the averages over bins b0..b1-1 of the nine sums per bin acc [bin][9][len]: phi,
// densities [species][len] and fluxes [species][3][len] (times wv), each if not null
void launch_avg_out(const double* acc, int b0, int b1, long len, const unsigned long long* cnt,
                    double wv, double* phi, double* n_out, double* flux_out, hipStream_t st);
// counting sort of the slots in use into dst (dropping empty slots, padding
// every tile to a multiple of 4), and the particles in MD cubes listed anew in
// md_list, *n_md of them; capacity bounds the slots in use
void launch_sort(const PartF64& src, const PartF64& dst, const WorkLists& L, const MdTables& md,
                 int nx, int ny, int32_t* md_list, int* n_md, int* hist, int* sums, long capacity,
                 hipStream_t st);
void launch_sort(const PartF32R& src, const PartF32R& dst, const WorkLists& L, const MdTables& md,
                 int nx, int ny, int32_t* md_list, int* n_md, int* hist, int* sums, long capacity,
                 hipStream_t st);
void launch_fill_int(int* a, long n, int v, hipStream_t st);
// the step's ionisations made into particles (one block; see ionize_kernel):
// exactly one of the FP64 and FP32R pointer pairs is non-null
void launch_ionize(const PartF64* Pe64, const PartF64* Pi64, const PartF32R* Pe32,
                   const PartF32R* Pi32, const WorkLists& Le, const WorkLists& Li,
                   const SpeciesStep& Se, const MdTables& md, uint32_t* next_id, long room_e,
                   long room_i, unsigned long long* dropped, hipStream_t st);
// FP64 energy diagnostic: per-block sums (energy_blocks() of them) of |v|^2
// over a species' live particles, and of |E|^2 times each node's share of a
// cell volume over the mesh (E as stored: double pairs if e_f64, else float4)
int energy_blocks();
void launch_energy(const PartF64* P64, const PartF32R* P32, const WorkLists& L, double* out,
                   hipStream_t st);
void launch_field_energy(const void* E, int e_f64, long nxy, int nz, double* out, hipStream_t st);

// mesh
// one grain's share of the right-hand side: interior node `node` (the index
// into b), grain g, its cloud-in-cell weight there (w, the FP64 form) and the
// fixed-point part of its charge quantum (part, FP32R); a replica's table is
// sorted by node, then by grain and corner
struct GrainShare {
  long long part;
  double w;
  int node;
  int g;
};
// The FP64 Poisson solve on the half spectrum (spectral.hip).  A line of
// length N: its radices, and per stage the multiplier that divides by the
// product of the earlier radices (see div_by).
constexpr int kFftStages = 8;
constexpr int kRowThreads = 1024;  // threads of a block that takes whole planes
struct FftLine {
  int N, nst;
  int radix[kFftStages];
  unsigned mul_s[kFftStages];
};
// hx = nx / 2 + 1 independent columns, npair row pairs, ldx the row stride of
// the packed rows in LDS (odd), buf elements per LDS buffer; full: a block
// takes a whole plane, else `pairs` row pairs (chunks of them a plane) and, in
// a kernel of their own, `cols` columns (col_chunks of them)
struct SpectralPlan {
  FftLine fx, fy;
  int K, hx, npair, ldx, buf, full;
  int pairs, chunks, cols, col_chunks;
  unsigned mul_nx, mul_hx, mul_pairs, mul_last, mul_cols, mul_cols_last;
};
// false if a side has a prime factor above 5
bool spectral_plan(int nx, int ny, int nz, SpectralPlan* p);
int spectral_setup();  // once per device before the first solve; 0 on success
// what the right-hand side is formed from: the unit charge of one grain, the
// FP64 accumulator, or the fixed-point one
enum { kRhsUnit = 0, kRhsRho64 = 1, kRhsFixed = 2 };
struct SpectralArgs {
  const double2 *tw_x, *tw_y;
  const double* rho64;
  const long long* rhofx;
  double scale;
  const GrainShare* tab;
  const int* tab_start;  // [blocks of the rows kernel + 1] first entry of each; null without grains
  int unit;
  const unsigned long long* counts;
  int ng;
  double we;
  double* Q;
  double* psi;  // the result, interior planes
  double* b;    // kRhsFixed: the right-hand side, stored
};
// The refinement's record (FP32R; ctl null: none): norms[0..1] ||r||^2 and
// ||b||^2 of the residual a solve ended with, ctl[0] whether it met the
// tolerance, ctl[1] sweeps, ctl[2] solves that did not, ctl[3] set while the
// last solve's sums (`partials`, nb pairs, from the field kernel) are still to
// be added up: the next solve does so on its way, or launch_final_test.
struct RefineState {
  const double* partials;
  int nb;
  double* norms;
  int* ctl;
  double tol2;
};
void launch_spectral_solve(const SpectralPlan& p, const SpectralArgs& a, int in, double2* work,
                           const double* inv, const RefineState& rs, hipStream_t st);
void launch_final_test(const RefineState& rs, hipStream_t st);
// tridiagonal factors of `cols` columns from sin^2 tables (pi m / nx, pi n / ny)
void launch_factors(const double* sx2, const double* sy2, int cols, int ny, int K, double* inv,
                    hipStream_t st);
void launch_solve_refined(const FftPlanHost& P, int nx, int ny, int nz, const double* b,
                          double* psi, double* r, void* work32, const void* tw_x32,
                          const void* tw_y32, const void* inv, int sweeps,
                          double tol, double* norms, int* ctl, hipStream_t st,
                          bool have_r0 = false);
// the FP32R right-hand side (fixed-point rho and the grains' shares, tab)
// and the first residual with its norm partials (partials = norms + 2 of the
// refined solve, which then runs with have_r0); also freezes Q_g
void launch_rhs_residual(const long long* rho, double scale, const GrainShare* tab, int ntab,
                         const unsigned long long* counts, int ng, double we, double* Q,
                         double* b, const double* psi, double* r, int nx, int ny, int nz,
                         double* partials, hipStream_t st);
// the arguments of the FP32R right-hand side (launch_rhs_residual's)
struct RhsArgs {
  const long long* rho;
  double scale;
  const GrainShare* tab;
  int ntab;
  const unsigned long long* counts;
  int ng;
  double we;
  double* Q;
};
// launch_rhs_residual + launch_solve_refined(..., have_r0 = true) in fewer
// kernels where the plane transforms fit in LDS (same phi, psi and Q; the
// norms' partial sums are grouped differently).  With defer_final the
// residual after the last sweep and its test are left to the caller where that
// path applies (returns true; launch_refine_final).
bool launch_rhs_solve_refined(const RhsArgs& a, const FftPlanHost& P, int nx, int ny, int nz,
                             double* b, double* psi, double* r, void* work32,
                             const void* tw_x32, const void* tw_y32, const void* inv,
                             int sweeps, double tol, double* norms, int* ctl, hipStream_t st,
                             bool defer_final);
// the residual after the last of `sweeps` refinement sweeps and its stopping
// test (norms, ctl as launch_solve_refined); psi and b unchanged since the solve
void launch_refine_final(int nx, int ny, int nz, const double* b, const double* psi, double* r,
                         int sweeps, double tol, double* norms, int* ctl, hipStream_t st);
// field and potential of the unit-charge solve (interior potential psi, both
// electrodes at 0) on grain g's MD cube: U[g][3][(2c+2)^3], Uphi[g][(2c+2)^3]
void launch_extract_cube(const double* psi, const int* gcell, int g, int c, int nx, int ny, int nz,
                         double dx, double* U, double* Uphi, hipStream_t st);
// the potential on the fine grid's nodes (stored, or added to the rf-phase
// bin of the step when avg.step is set); Uphi may be null without grains
void launch_fine_phi(const double* phi, const MdTables& md, const double* Uphi, const FineBox& fb,
                     int nx, int ny, int nz, double dx, double radius, double* out,
                     const AvgBins& avg, hipStream_t st);
void launch_e_out(const double* E64, const float* E32, double* out, long nn, hipStream_t st);
// the total charge density: conv * (plasma + grains), or that sum in fixed point (outfx)
void launch_rho_out(const double* acc64, const long long* accfx, const GrainShare* tab, int n_tab,
                    const unsigned long long* counts, double conv, double* out, long long* outfx,
                    long plane, long nn, hipStream_t st);
// moments [species][4][nn] times conv into the densities [species][nn] and the
// fluxes [species][3][nn] (either may be null)
void launch_moments_out(const double* mom, long nn, double conv, double* n_out, double* flux_out,
                        hipStream_t st);
void launch_scale(double conv, double* a, long n, hipStream_t st);
void launch_zero_f64(double* a, long n, hipStream_t st);
void launch_zero_i64(long long* a, long n, hipStream_t st);
void launch_zero_i32(int* a, long n, hipStream_t st);

}  // namespace pic
