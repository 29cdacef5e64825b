// Internal declarations shared by the kernel file and the host library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <memory>
#include <vector>

#include "../../include/fsv.h"

namespace fsv {

// One excitation rotation compiled for the dense kernels.  The active source
// strings are base | src and their partners base | dst, where base has zeros
// at the nt sorted target qubits q[]; the JW sign of tau on the source is
// sign0 * (-1)^popcount(base & par).
struct RotOp {
    uint64_t src, dst, par;
    uint32_t q[4];
    int32_t nt;
    int32_t sign0;
};

// One excitation on the sector-compressed state C[Ia][Ib] (alpha-string-first
// product basis = blocked JW ordering restricted to the sector).  Its active
// pairs are the product of an alpha pair list and a beta pair list; a list
// length of -1 means "every string maps to itself with sign +1".  List entries
// pack the source string (bits 0..14), the partner (15..29) and a negative-sign
// flag (bit 31); the pair sign is sign0 times both flags.
struct PairOp {
    int32_t nA, nB;
    int64_t offA, offB;
    int32_t sign0, pad;
};

__host__ __device__ inline uint32_t pack_pair(uint32_t s, uint32_t d, int neg) {
    return s | (d << 15) | (neg ? 0x80000000u : 0u);
}

// Launch shape of the pair kernels.
struct Shape {
    int block;   // threads per workgroup
    int ppt;     // pairs per thread per loop trip (1, 2, 4, 8)
};

// Packed string excitation: bits 0..15 source string J, 16..24 p*M+q,
// bit 31 set for a negative sign.
__host__ __device__ inline uint32_t pack_exc(uint32_t J, uint32_t pq, int neg) {
    return J | (pq << 16) | (neg ? 0x80000000u : 0u);
}

// ---- host helpers shared by plans and batches (fsv_host.hip) ----
int fail(int code, const char *fmt, ...);
void clear_error();
// True when every operation queued on st has completed.  A query that fails
// for any other reason counts as pending, so that the caller fences.
inline bool stream_idle(hipStream_t st) {
    const hipError_t q = hipStreamQuery(st);
    if (q == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}
int validate_problem(const fsv_problem *p);
int validate_ops(int n_qubits, int n_ops, const int32_t *ops);
// excitation 1: a qubit excitation (no JW string: sign +1 on every pair)
RotOp compile_op(int M, int ordering, const int32_t *op, int excitation = 0);
std::vector<uint32_t> strings_of(int M, int N);  // popcount-N masks, ascending
// Prefix-parity mask of a beta string b (M spatial orbitals) for a qubit
// ordering (0: qubit 2p + s, 1: qubit p + s M): bit q is set when an odd
// number of b's occupied beta orbitals sit on qubits below alpha orbital q's
// qubit.  (-1)^popcount(a & mask) is the sign between the qubit-basis
// amplitude of determinant (a, b) and its alpha-first sector amplitude.
uint32_t beta_prefix_parity(int M, int ordering, uint32_t b);
void build_string_h(int M, const std::vector<uint32_t> &str, const std::vector<int32_t> &rank,
                    const double *ht, const double *g, std::vector<int64_t> &ptr,
                    std::vector<int32_t> &col, std::vector<double> &val);
// Per string (ascending rank): its excitations p -> q, q empty, then its
// diagonal entries p -> p (the last popcount entries), as packed words.
void build_exc(int M, const std::vector<uint32_t> &str, const std::vector<int32_t> &rank,
               std::vector<uint32_t> &exc, int &nexc);
// Partner table of the row kernels (SectorTabs::tp) for the strings of one spin.
std::vector<uint32_t> build_partners(int M, const std::vector<uint32_t> &str, const std::vector<int32_t> &rank);
// Per string: the factor rows Lt[pp][0..rp) of its occupied p summed (its
// diagonal excitations folded into one), nstr x rp.
std::vector<double> diag_factor_sums(int M, const std::vector<uint32_t> &str, const std::vector<double> &Lt, int rp);
// Pivoted Cholesky of a symmetric positive semidefinite n x n matrix:
// G ~ sum_k L_k L_k^T with R rows of L (length n); returns R, or -1 when G is
// not positive semidefinite within tol * max(diag).
int pivoted_cholesky(int n, const double *G, double tol, std::vector<double> &L);
// Pair lists of one operator for the sector-compressed state; appends to lists.
PairOp build_pair_op(int M, const int32_t *op, const std::vector<uint32_t> &sa,
                     const std::vector<int32_t> &ra, const std::vector<uint32_t> &sb,
                     const std::vector<int32_t> &rb, std::vector<uint32_t> &lists);
// The same for a qubit excitation in the given qubit ordering.
PairOp build_pair_op_qeb(int M, int ordering, const int32_t *op, const std::vector<uint32_t> &sa,
                         const std::vector<int32_t> &ra, const std::vector<uint32_t> &sb,
                         const std::vector<int32_t> &rb, std::vector<uint32_t> &lists);

// ---- launchers (fsv_kernels.hip) ----
// precision: 0 complex128, 1 complex64.  Each returns the hipError_t of the launch.
int max_grid();
void init_kernels();  // once per process, before any capture (sets kernel attributes)

hipError_t launch_fill_zero(void *ptr, size_t bytes, hipStream_t st);
hipError_t launch_set_amp(void *psi, int vtype, uint64_t x, double re, hipStream_t st);
hipError_t launch_copy_doubles(const double *src, double *dst, int n, hipStream_t st);
// psi[idx[i]] = (val[i], 0) for i < n; vtype selects the storage (VType).
hipError_t launch_set_list(void *psi, int vtype, const int64_t *idx, const double *val, int n, hipStream_t st);

// Grid used for op with npairs pairs under shape sh (fixed per op: reductions
// depend on it).
unsigned rot_grid(uint64_t npairs, Shape sh);

hipError_t launch_rot(int precision, bool wide, void *psi, const RotOp &op, const double *cs,
                      int k, uint64_t npairs, Shape sh, hipStream_t st);
hipError_t launch_adj(int precision, bool wide, void *psi, void *lam, const RotOp &op,
                      const double *cs, int k, uint64_t npairs, Shape sh, double *partial,
                      hipStream_t st);
// LDS-staged fused run: ops [k0, k1) whose targets all lie below tile_bits are
// applied block by block in one pass over psi (+theta in order).
hipError_t launch_rot_fused(int precision, void *psi, const RotOp *ops_dev, const double *cs,
                            int k0, int k1, int tile_bits, uint64_t n_amps, hipStream_t st);
// Its adjoint: one pass over psi and lam undoes ops k1-1 .. k0 and writes each
// operator's gradient partials to partial[k * pstride + b], b < fused_grid().
// At most max_fused_run() operators.
hipError_t launch_adj_fused(int precision, void *psi, void *lam, const RotOp *ops_dev, const double *cs,
                            int k0, int k1, int tile_bits, uint64_t n_amps, double *partial, int pstride,
                            hipStream_t st);
unsigned fused_grid(uint64_t n_amps, int tile_bits);
int max_fused_run();

// out[0] = the energy partials' sum, out[1 + k] = 2 x operator k's gradient
// partials' sum (rows as in launch_reduce_rows), one launch; host (pinned,
// coherent) receives the same k + 1 values.
hipError_t launch_reduce_eg(const double *epart, const int *ecount, const double *gpart, const int *gcount,
                            int stride, int k, double *out, double *host, hipStream_t st);
hipError_t launch_reduce_rows(const double *partial, const int *counts, int stride, int rows,
                              double scale, double *out, hipStream_t st);

// Complex sector states as planes: row Ia holds nsb real, then nsb imaginary
// parts.  *im_flag = im_epoch when an imaginary part is not zero.
hipError_t launch_gather(int precision, const void *psi, const uint64_t *Xa, const uint64_t *Xb,
                         const uint32_t *sa, const uint32_t *PPb, int64_t nsa, int64_t nsb,
                         double *C, int32_t *im_flag, int32_t im_epoch, hipStream_t st);
hipError_t launch_scatter(int precision, void *lam, const double *S, const uint64_t *Xa,
                          const uint64_t *Xb, const uint32_t *sa, const uint32_t *PPb,
                          int64_t nsa, int64_t nsb, hipStream_t st);
hipError_t launch_rdm_overlap(const double *A, int64_t nrows, int64_t ncols,
                              const uint32_t *exc, int nexc, const int32_t *im_flag, int32_t im_epoch,
                              double2 *O, hipStream_t st);
hipError_t launch_rdm_bin(const double2 *O, const int32_t *off, const int32_t *idx, int nbins,
                          double2 *out, hipStream_t st);

// ---- sector-compressed kernels (fsv_sigma.hip) ----
// Amplitude storage of a compact sector vector.
enum VType { V_C128 = 0, V_C64 = 1, V_F64 = 2, V_F32 = 3 };
inline int vtype_bytes(int vt) { return vt == V_C128 ? 16 : (vt == V_F32 ? 4 : 8); }

// Device tables of one sector Hamiltonian (alpha-first basis).
struct SectorTabs {
    int64_t nsa, nsb;
    int M, nexcA, nexcB;
    const int64_t *ha_ptr, *hb_ptr;
    const int32_t *ha_col, *hb_col;
    const double *ha_val, *hb_val;
    const uint32_t *excA, *excB;
    const double *g;
    double ecore;
    // Optional exact factorisation (pq|rs) = sum_l L[l][pq] L[l][rs] of rank R
    // (pivoted Cholesky of the pair supermatrix): Lt holds L transposed and
    // padded to 8 columns (M^2 x 8, zero beyond R).  R = 0 (also for every
    // rank above 8): direct product.
    int R;
    const double *Lt;
    // Optional dense same-spin string Hamiltonians applied as FP64 GEMMs
    // through the rocBLAS handle blas (alpha row-major; beta transposed, added
    // into S, not used with the factorisation); nullptr: the CSR rows above.
    const double *ha_dense, *hb_dense_t;
    void *blas;
    // Each string's list in excA / excB ends with its ndA (ndB) diagonal
    // entries p -> p.  With the factorisation, da: per alpha string the factor
    // rows of its diagonal excitations summed (nsa x 8); db: the same per beta
    // string, one row per factor (8 x 2 ceil(nsb / 2)).
    int ndA, ndB;
    const double *da, *db;
    // Partner table of the beta strings for the row kernels: orbital pairs p <
    // q in lexicographic order, then the diagonal ones p = p; per pair ts =
    // ceil(nsb / 2) words, word j the partners of strings 2 j and 2 j + 1 in
    // 16 bits each: the rank, 2 ts + 2 more for a negative sign, or 2 ts where
    // the pair does not reach the string.
    const uint32_t *tp;
    // Factors of the off-diagonal pairs (pairs x 8), and the one-body values
    // h' = h + v - 1/2 sum_r (pr|rq): all of them (M x M), per off-diagonal
    // pair, and summed over each string's occupied orbitals.
    const double *Lp, *heff, *hp, *hda, *hdb;
    // Direct product: (pq|rs) with rs packed in the order of tp (M^2 x npp,
    // zero beyond the pairs), and per alpha string its diagonal rows summed
    // (nsa x npp); nullptr: rows that k_abm and k_ab do not take.
    const double *gp, *dg;
    int npp;
};

int cadj_blocks(const PairOp &op, int64_t nsa, int64_t nsb);  // partials written by launch_cadj
hipError_t launch_crot(int vtype, void *psi, const PairOp &op, const uint32_t *lists,
                       const double *cs, int k, int64_t nsa, int64_t nsb, hipStream_t st);
hipError_t launch_cadj(int vtype, void *psi, void *lam, const PairOp &op, const uint32_t *lists,
                       const double *cs, int k, int64_t nsa, int64_t nsb, double *partial,
                       hipStream_t st);
// Real sector states (V_F64 / V_F32) only: z[i] = (psi[i], lam[i]) for i < n,
// and launch_cadj on such interleaved pairs.
hipError_t launch_zip(int vtype, const void *psi, const void *lam, void *z, int64_t n, hipStream_t st);
hipError_t launch_cadj_zip(int vtype, void *z, const PairOp &op, const uint32_t *lists, const double *cs, int k,
                           int64_t nsa, int64_t nsb, double *partial, hipStream_t st);
// out (vtype_out) <- in (vtype_in), element-wise; complex <-> real keeps the real part.
hipError_t launch_convert(int vt_in, const void *in, int vt_out, void *out, int64_t n, hipStream_t st);
// S = H C on the sector.  planes = 1: real states, nsa x nsb; planes = 2:
// complex ones, nsa rows of nsb real then nsb imaginary parts.  CT, ST: work
// arrays of the same size.  Writes sigma_partials(T, planes) partials of
// Re<C|S>.  zout (real states, may be null): where the product's last step
// allows it, the (C, S) pairs go to zout (of type zvt) instead of S, and
// *zipped is set.
unsigned combine_grid(int64_t dim);
int sigma_partials(const SectorTabs &T, int planes);
// Whether rows of ncols columns fit k_row (factorised) and k_abm or k_ab (direct).
bool row_kernel_fits(int64_t ncols);
bool ab_kernel_fits(int64_t ncols);
hipError_t launch_sector_sigma(int planes, const SectorTabs &T, const double *C, double *S, double *CT,
                               double *ST, double *epart, hipStream_t st, void *zout = nullptr, int zvt = V_F64,
                               bool *zipped = nullptr);
// Only the partials of Re<C|H|C>; S, CT, ST are work arrays.  planes = 2: the
// imaginary parts may be taken as zero unless *im_flag equals im_epoch.
hipError_t launch_sector_energy(int planes, const SectorTabs &T, const double *C, double *S, double *CT,
                                double *ST, double *epart, const int32_t *im_flag, int32_t im_epoch,
                                hipStream_t st);
// hp, hda, hdb of the row kernels from h' (strings sa, sb as masks).
hipError_t launch_row_onebody(const double *heff, int M, const uint32_t *sa, int64_t nsa, const uint32_t *sb,
                              int64_t nsb, double *hp, double *hda, double *hdb, hipStream_t st);
// ADAPT pool screening on a real sector state (V_F64 / V_F32): grid (gx, n_ops),
// partial[t * gx + x] = workgroup x's share of Re<lam|T_t|psi> for pool op t.
hipError_t launch_pool(int vtype, const void *psi, const void *lam, const PairOp *ops, const uint32_t *lists,
                       int n_ops, int gx, int64_t nsa, int64_t nsb, double *partial, hipStream_t st);
// Screening by rows.  A group holds the pool operators (gops[op0 ...], ngen
// with a beta list, then nplain without one) that share the row pairs at
// lists[offA ...] (offA = -1: every row with itself); its tasks (group, first
// row pair) take U row pairs each (kPoolU in groups with ngen = 0, whose tasks
// come last), and operator t's partials (chunks x parts, one part for plain
// operators) start at partial[off[t]].
constexpr int kPoolU = 4;
struct PoolGroup {
    int32_t op0, ngen, nplain, nA, parts, pad;
    int64_t offA;
};
// U for a pool of so many amplitude pairs in all its operators and row pairs in all
// its groups; 0: the pool is screened operator by operator (launch_pool).
int pool_rows_u(int vtype, int64_t nsa, int64_t nsb, double pairs, double rows);
hipError_t launch_pool_rows(int vtype, const void *psi, const void *lam, const PairOp *ops, const uint32_t *lists,
                            const PoolGroup *groups, const int32_t *gops, const int2 *tasks, int n_gen, int n_plain,
                            int U, int64_t nsb, const int64_t *off, double *partial, int n_ops, double *out,
                            hipStream_t st);
// String Hamiltonian values val[e] = v2[e] + one-body part of descriptor
// desc[e] with h~ = ht (M x M): -1 none, -2 - I the diagonal of row I (sum of
// h~_ii over the occupied orbitals of string str[I]), otherwise h~[desc &
// 0x3FFFFFFF], negated when bit 30 is set.
hipError_t launch_string_h_values(double *val, const double *v2, const int32_t *desc, const uint32_t *str,
                                  const double *ht, int M, int64_t n, hipStream_t st);
// Dense row-major copy (n x n) of an n-row CSR matrix.
hipError_t launch_csr_dense(const int64_t *rowptr, const int32_t *col, const double *val, double *out, int64_t n,
                            hipStream_t st);
// Transpose of each plane of a compact vector: row r of `in` holds planes x
// cols values, row c of `out` planes x rows.
hipError_t launch_plane_transpose(const double *in, double *out, int64_t rows, int64_t cols, int planes,
                                  hipStream_t st);
// Real compact vector (double) -> dense complex buffer of 2^n amplitudes, all of
// them written.  ra, rb: per string mask of n/2 bits the string's rank or -1 (rb:
// and its prefix parity).
hipError_t launch_dense_image(int precision, int ordering, void *out, const double *S, const int32_t *ra,
                              const int2 *rb, int n, int na, int nb, int64_t nsb, hipStream_t st);
void init_sigma_kernels();  // by init_kernels only

// ---- fused operator runs on the sector state (fsv_fused.hip, fsv_packet.hip) ----
constexpr int kPacketAmps = 256;  // amplitudes (index slots) of one packet
// A run of consecutive operators applied tile by tile in LDS (fused = 1), by
// connected-component packets (fused = 2), a whole sweep in one workgroup
// (fused = 3, launch_whole), or a single operator left to the per-operator
// kernels (fused = 0, nops = 1).  A tile run keeps, per alpha
// orbit, a program of astride words (row count, row ranks, per-operator local
// alpha pairs) and, per beta block, one of bstride words (first column, width,
// per-operator local beta pairs).  A packet run keeps n_packets index lists
// (at ent_off, 256 words each) and regions of wr words (at reg_off).
struct FGroup {
    int32_t k0, nops, fused;
    int32_t n_orbits, n_blocks;  // tiles = n_orbits x n_blocks
    int32_t rmax, lmax;          // largest orbit (rows) and block (columns)
    int32_t astride, bstride;
    int64_t aprog_off, bprog_off;
    size_t lds;                  // dynamic LDS bytes of one tile / packet workgroup
    int32_t n_packets, wr;
    int64_t ent_off, reg_off;
    // Forward sweep from the reference state: while the state is zero outside
    // a few components, only the packets that hold nonzero amplitudes need to
    // run.  sub_n >= 0: those packets' programs, copied contiguously at
    // sub_ent_off / sub_reg_off; -1: launch every packet.
    int32_t sub_n = -1;
    int64_t sub_ent_off = 0, sub_reg_off = 0;
};

struct FusedOpts {
    size_t budget = 65536;       // LDS bytes of tile data per workgroup
    size_t lds_limit = 65536;    // dynamic LDS a workgroup may use
    int es = 8;                  // bytes per stored amplitude
    int arrays = 1;              // 1: forward (psi); 2: adjoint (psi and lam)
    int mode = 0;                // 0 fuse where the cost model gains, 1 never, 2 every run of >= 2
    int cus = 256;               // compute units (tiles resident at once scale with it)
    int min_block = 32;          // columns per block when blocks are split for more tiles
    int max_ops = 32;            // operators per run
    int64_t max_tiles = 8192;    // tiles per run (gradient partial slots per operator)
    bool place_xcd = true;       // packet runs: place components by XCD (padding with empty packets)
};

struct FusedSched {
    std::vector<FGroup> groups;  // in operator order
    std::vector<int> count;      // per operator: gradient partials of its fused run, -1 if not fused
    uint32_t *d_aprog = nullptr, *d_bprog = nullptr;  // packet runs: index lists, regions
    bool packets = false;        // built by build_packets: the adjoint sweep runs on (psi, lam) pairs
    std::vector<std::shared_ptr<void>> mem;  // device buffers (shared by schedules that alias them)
    size_t bytes = 0;                        // their size
    void release();
    void share(const FusedSched &o) {  // the same runs and device tables as o
        release();
        groups = o.groups;
        count = o.count;
        d_aprog = o.d_aprog;
        d_bprog = o.d_bprog;
        packets = o.packets;
        mem = o.mem;
        bytes = o.bytes;
    }
    FusedSched() = default;
    FusedSched(const FusedSched &) = delete;
    FusedSched &operator=(const FusedSched &) = delete;
    ~FusedSched() { release(); }
};

// Runs and tiles for the operators (K x 4 spin-orbital labels in ops, their
// pair ops and host pair lists) under o.  Returns an FSV_ status.
int build_fused(int M, const std::vector<uint32_t> &sa, const std::vector<uint32_t> &sb,
                const std::vector<PairOp> &pops, const std::vector<uint32_t> &lists,
                const std::vector<int32_t> &ops, const FusedOpts &o, FusedSched &S);
int fused_runs(const FusedSched &S, int *n_fused_ops);
// Host side of packet runs: groups (fused = 2 for packet runs, 0 for
// operators left alone), per-operator partial counts, and the index lists and
// regions (FGroup::ent_off / reg_off index ent / reg).  every_run: every run,
// a single operator's included, becomes a packet run.
struct PacketPlan {
    std::vector<FGroup> groups;
    std::vector<int> count;
    std::vector<uint32_t> ent, reg;
};
int plan_packets(int64_t nsa, int64_t nsb, const std::vector<PairOp> &pops, const std::vector<uint32_t> &lists,
                 const FusedOpts &o, bool every_run, PacketPlan &S);
// Batched packet runs over independent instances (real FP64 states in one
// arena): launch r carries run r - (R - runs_i) of every instance i (runs
// aligned at the end, so the adjoint sweep runs the same launches backwards).
struct BatchPacketInst {
    int64_t nsa, nsb, off_state, off_ops, off_k;
    int32_t K;
};
struct BatchPackets {
    int runs = 0;
    int pstride = 1;                       // gradient partial slots per operator
    std::vector<int64_t> ent_off, reg_off;  // per launch
    std::vector<int32_t> wr, npk;           // per launch: region stride, packets
    std::vector<uint32_t> ent, reg;
    std::vector<int32_t> count;             // per operator (global index): partials of its run
};
int build_batch_packets(const std::vector<BatchPacketInst> &insts, const std::vector<PairOp> &ops,
                        const std::vector<uint32_t> &lists, BatchPackets &B);
size_t batch_packet_lds(int wr, bool adjoint);
hipError_t launch_batch_packets(bool adjoint, double *arena, const uint32_t *ent, const uint32_t *reg, int wr,
                                int npk, const double *cs, double *gpart, int pstride, hipStream_t st);

// Packet runs (fused = 2) for sector states of at most packet_max_dim()
// amplitudes; o.es, o.mode (0 cost model, 1 never, otherwise every run of >= 2)
// and o.max_ops are used.  count[k] = gradient partials of operator k's run.
// Plans use them by default up to packet_default_dim() amplitudes (above it
// only on request: planning time and program memory grow with the state).
int64_t packet_max_dim();
int64_t packet_default_dim();
int build_packets(int64_t nsa, int64_t nsb, const std::vector<PairOp> &pops, const std::vector<uint32_t> &lists,
                  const FusedOpts &o, FusedSched &S);
// One packet run: forward (state = psi) or adjoint (state = the interleaved
// (psi, lam) pairs of launch_zip; gradient partials gpart[k * gstride + workgroup]).
// t0, t1 (optional): events given the kernel's own start and end times.
// store = false: the run's results are not written back (nothing reads them:
// the adjoint sweep's last run).
hipError_t launch_packets(int vtype, bool adjoint, void *state, const FusedSched &S, const FGroup &g,
                          const double *cs, double *gpart, int gstride, hipStream_t st, hipEvent_t t0 = nullptr,
                          hipEvent_t t1 = nullptr, bool store = true);
// A whole sweep in one workgroup (fused = 3: rmax steps, wr threads, lmax
// amplitudes) for states of at most whole_max_dim(bytes per amplitude)
// amplitudes.  Forward: initialises the state itself (n entries idx / val, or
// the amplitude ref at index 0) and writes psi; adjoint: reads the (psi, lam)
// pairs and writes only gradient partials.
struct WholeInit {
    int32_t n = 0;
    const int64_t *idx = nullptr;
    const double *val = nullptr;
    double ref = 1.0;
};
int64_t whole_max_dim(int es);
int build_whole(int64_t nsa, int64_t nsb, const std::vector<PairOp> &pops, const std::vector<uint32_t> &lists, int es,
                FusedSched &S);
hipError_t launch_whole(int vtype, bool adjoint, void *state, const FusedSched &S, const FGroup &g, const double *cs,
                        const WholeInit &in, double *gpart, int gstride, hipStream_t st);
void init_fused_kernels();  // by init_kernels only
size_t fused_lds_limit();
// Forward (psi) or adjoint (psi, lam, gradient partials gpart[k * gstride + tile]).
// Packet groups are launched with launch_packets.
hipError_t launch_fused(int vtype, bool adjoint, void *psi, void *lam, const FusedSched &S, const FGroup &g,
                        const PairOp *d_pops, const double *cs, int64_t nsb, double *gpart, int gstride,
                        hipStream_t st);

}  // namespace fsv
