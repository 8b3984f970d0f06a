// Internal declarations shared by the translation units of libdrf.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <math.h>
#include <string>
#include <vector>

#include "../../include/drf.h"

namespace drf {

// ---- errors -----------------------------------------------------------------
void set_error(const char* fmt, ...);
#define DRF_FAIL(code, ...) do { ::drf::set_error(__VA_ARGS__); return (code); } while (0)
#define DRF_HIP(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) { \
    ::drf::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
    return DRF_EHIP; } } while (0)

// ---- schedule / plan (host) ---------------------------------------------------
struct Schedule {
    std::vector<double> abar;   // cumulative alpha per training timestep
    int steps = 0, stride = 0, train_steps = 0;
    drf_sampler sampler = DRF_DDIM;
    double eta = 0.0, shift = 1.0;
    int tau(int s) const { return (s - 1) * stride; }
    double abar_at(int s) const { return s == 0 ? 1.0 : abar[(size_t)tau(s)]; }
    // Euler: ODE time of sampling index s
    double sigma_at(int s) const;
    // integer time fed to the network at sampling index s >= 1
    int net_time(int s) const;
    // true when some transition of this sampler adds fresh noise
    bool stochastic() const { return sampler == DRF_DDPM || (sampler == DRF_DDIM && eta != 0.0); }
    // x_to = A x_from + B net + C z.  Fails for a transition with variance that is not a move towards data.
    drf_status coef(int s_from, int s_to, float* A, float* B, float* C) const;
};
drf_status make_schedule(const drf_sched_config* sc, Schedule* out);

// One batched predictor pass of drf_sample and the elementwise update after it.
struct Pass {
    int round = 0;
    bool solo = false;              // stand-alone evaluation of the anchor state
    int s_anchor = 0;               // anchor index the evaluated states were drafted from
    std::vector<int> eval_s;        // sampling indices evaluated, one per slot group
    bool base_is_draft = false;     // chain starts from the first draft, else from the anchor state
    std::vector<std::pair<int, int>> chain;   // standard updates (s_from -> s_to); update i uses noise field i
    std::vector<int> chain_z;       // per update: ordinal of its fresh-noise field among the call's draws
    int anchor_field = -1;          // noise field that pairs with the state after the chain (-1: none)
    std::vector<int> draft_to;      // skip targets drafted from (state after chain, anchor noise)
    std::vector<int> draft_z;       // per draft: ordinal of its fresh-noise field
    int s_after = 0;                // index of the state after the chain
    bool writes_x0 = false;         // the state after the chain (or the lone draft to 0) is x_0
};
// rows: plan table in the documented row format (may be NULL).  n_noise (may be NULL): number of
// fresh-noise fields the call draws (kind-1 plus kind-2 rows).
drf_status build_plan(const Schedule& sch, drf_mode mode, int n, std::vector<Pass>* passes,
                      std::vector<int32_t>* rows, size_t* n_noise = nullptr);

// ---- elementwise update kernel --------------------------------------------------
constexpr int kMaxBlock = 64;       // largest block size n the update kernel's argument block holds
struct UpdateArgs {
    const float* x_base;   // [field]
    const float* eps;      // [n_fields][g][field]
    float* x_out;          // [field] or NULL: state after the chain
    float* draft_out;      // [n_draft][field] or NULL
    size_t field;          // batch * elems_per_sample
    int g;                 // 1, or 2 = (cond, null) pairs combined by guidance
    float w;               // guidance scale
    int n_chain, anchor_field, n_draft;
    float cA[kMaxBlock], cB[kMaxBlock], dA[kMaxBlock], dB[kMaxBlock];
    // fresh noise: y += cC[i] * z(field cz[i]) after chain update i, d_j += dC[j] * z(field dz[j]);
    // a zero coefficient means the field is not touched
    int noise_mode;        // 0 none | 1 explicit fields at z | 2 generated from (seed, z_field0 + ordinal)
    const float* z;        // [..][field]
    uint64_t seed;
    uint32_t z_field0;
    float cC[kMaxBlock], dC[kMaxBlock];
    int cz[kMaxBlock], dz[kMaxBlock];
};
enum { NOISE_NONE = 0, NOISE_EXPLICIT = 1, NOISE_PHILOX = 2 };
// Fills noise_mode / z / seed / z_field0 from the caller's source; fails when a nonzero cC / dC has no source.
drf_status set_noise_source(UpdateArgs* a, const drf_noise* noise);
drf_status launch_update(const UpdateArgs& a, hipStream_t st);

// ---- DiT kernels ------------------------------------------------------------------
typedef __bf16 bf16_t;

// How slot j of a pass finds its inputs.
struct SlotMap {
    const int32_t* t_dev;   // per-slot training timesteps, or NULL: use taus[j / group]
    int group;              // slots per draft group (g * batch)
    int taus[kMaxBlock];
    int x_group, x_batch;   // x row of slot j = (j / x_group) * x_batch + j % x_batch
    int cond_mod;           // cond row of slot j = cond_mod ? j % cond_mod : j
};

enum EpiMode { EPI_STORE = 0, EPI_STORE_GELU = 1, EPI_RESID = 2, EPI_STORE_HEADS = 3, EPI_STORE_GATED = 4,
               EPI_STORE_SILU = 5 /* fp32 path only */ };
__device__ inline float silu(float v) { return v / (1.f + __expf(-v)); }
struct Epilogue {
    int mode;
    void* out;              // EPI_STORE*: [M][ldo] of out type; EPI_RESID: float [M][ldo], read-modify-write
    int ldo;
    int out_f32;            // EPI_STORE*: 1 = float output, 0 = bf16 output
    const float* bias;      // [N]
    const float* gate;      // EPI_RESID, EPI_STORE_GATED: gate[(m / rows_per_slot) * gate_ld + n]; EPI_RESID: NULL = ungated
                            // EPI_STORE_GATED (bf16 only): out = gate * (acc + bias), the branch output that the next
                            // LayerNorm launch adds to the residual stream
    int gate_ld, rows_per_slot;
    uint32_t rps_magic; int rps_shift;   // m / rows_per_slot == fast_div(m, rps_magic, rps_shift), see set_rows_per_slot
    // EPI_STORE_HEADS (bf16 only): column n = which * hid + head * hd + dd of row m = slot * rows_per_slot + t goes to
    //   out[which * plane + ((slot * heads + head) * rows_per_slot + t) * hd + dd]     (q | k | v planes, head-major)
    // with the q plane multiplied by q_scale before it is rounded
    int hid, hd, heads; size_t plane; float q_scale;
    uint32_t hid_magic, hd_magic; int hid_shift, hd_shift;
    // Optional (bf16 kernels): the last 256 workgroups of the launch (the ones that run in its final round) each ask for
    // their share of the warm_lines 128-byte lines at `warm`, typically the weights of the GEMM that runs next, so that
    // those are already on the near side of HBM when that GEMM asks for them (see warm_caches in gemm_device.h).
    const void* warm; uint32_t warm_lines;
};
// Division constants for floor(n / d), 0 <= n < 2^31 (see fast_div in gemm_device.h).
void make_fast_div(int d, uint32_t* magic, int* shift);
// Fills rows_per_slot and its division constants (exact for 0 <= m < 2^31).
void set_rows_per_slot(Epilogue* e, int rows_per_slot);
// Partial tiles of a split-K launch that its consumer adds itself: element (m, n) of the product is
// sum over s < splits of part[s * stride + m * ldp + n].  splits == 0: there are none, the launch has stored its result.
constexpr int kMaxSplits = 6;       // parts that the choice of tile makes at most
struct PartialSum { const float* part; int splits, ldp; size_t stride; };
// How variant 0 of the launch below runs: `tile` (a number of kTiles in gemm.hip) with K in `splits` parts, the first
// first_rows rows (0: none) ahead of the others with first_tile.
struct GemmRoute { int tile, splits, first_tile, first_rows; };
GemmRoute gemm_route(int M, int N, int K, const Epilogue& e, bool may_split, bool leave);
// C[M][N] = A[M][K] . W[N][K]^T, then the epilogue.  bf16: K % 64 == 0.
// variant 0: the tile shape and split are chosen from the problem size; > 0 forces one (measurement and tile tests).
// splitk_scratch: gemm_splitk_scratch_bytes() of device memory, or NULL; with it, problems of few tiles and a long
// K may be split across workgroups (variant 10 forces the 128 x 128 tile, split when K is long enough; variant
// 100 s + v forces tile v split in s).
// leave != NULL: a launch that splits leaves its partial tiles for the caller (in splitk_scratch, the epilogue not applied).
drf_status launch_gemm_bf16(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st,
                            int variant = 0, float* splitk_scratch = nullptr, PartialSum* leave = nullptr);
// The 256-row tiles of 288 and of 256 columns on rows m_first .. M - 1; called by launch_gemm_bf16, which checks the shapes
// (no GELU with fp32 output).
drf_status launch_gemm_wide_288(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first);
drf_status launch_gemm_wide_256(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first);
drf_status launch_gemm_wide_192(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first);
drf_status launch_gemm_wide_192x288(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first);
// The tiles of gemm_pair.h (8, 13, 16, 17) on rows m_first .. M - 1, likewise.
drf_status launch_gemm_pair(int tile, const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first);
size_t gemm_splitk_scratch_bytes();
// fp32; a_row_mod: row m of C uses row m % a_row_mod of A (0: row m).
drf_status launch_gemm_f32(const float* A, const float* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int a_row_mod = 0);
// fp32, with LayerNorm and modulation of the rows of A computed on the way (K is the row length):
// A = (x - mean) / sqrt(var + 1e-6) * (1 + scale) + shift of row m's slot; shift NULL: no modulation.
struct RowNorm { const float *shift, *scale; int mod_ld, rows_per_slot; };
bool gemm_f32_folds_ln(int M, int N, int K);       // whether that is the faster way (and one that the launch takes)
drf_status launch_gemm_f32_ln(const float* resid, const RowNorm& ln, const float* W, int M, int N, int K, const Epilogue& e, hipStream_t st);

struct AttnArgs {
    // query i of (slot, head h) starts at q + slot * q_slot_stride + h * q_head_stride + i * ldq  (elements);
    // key/value j at k|v + kv_batch * kv_batch_stride + h * kv_head_stride + j * ldk.
    // Packed rows [row][.. head h at column h*d ..]: slot stride N * ld, head stride d.
    // Head-major [slot][head][row][d]: slot stride heads * N * d, head stride N * d, ld = d.
    const void* q; int ldq; size_t q_slot_stride, q_head_stride;
    const void* k; const void* v; int ldk; size_t kv_batch_stride, kv_head_stride;
    void* out; int ldo;             // out row (slot * Nq + i), head h at column h * d
    int Nq, Nk, heads, d, slots;
    int kv_mod;                     // kv_batch = kv_mod ? slot % kv_mod : slot
    int q_scaled;                   // bf16 path: 1 = the queries have been multiplied by log2(e) / sqrt(d) already
};
// Factor that turns q . k into an exponent of two.
inline float attn_scale_log2(const AttnArgs& a) { return a.q_scaled ? 1.f : 1.4426950408889634f / sqrtf((float)a.d); }
// Which bf16 kernel takes a launch (see attn_route in attn.hip for the rules).
enum AttnRoute {
    ATTN_SHORT = 1,         // up to 256 kv rows, one wave per 64 of them; 32 queries per workgroup (attn_short.hip)
    ATTN_SHORT_64 = 2,      // the same with 64 queries
    ATTN_CHUNKED = 3,       // chunks of kv rows, 8 waves of 32 queries, up to 256 kv rows (attn.hip)
    ATTN_CHUNKED_PERSIST = 4,   // the same, persistent workgroups
    ATTN_CHUNKED_LONG = 5,  // 8 waves, more than 256 kv rows
    ATTN_CHUNKED_FEW = 6,   // 4 waves, up to 128 queries
    ATTN_LONG = 7,          // more than 256 kv rows, or more than 256 queries over fewer: 64 queries per wave (attn_long.hip)
};
AttnRoute attn_route(int Nq, int Nk, int heads, int d, int slots, bool q_scaled);
// Self-attention whose queries their producer should multiply by log2(e) / sqrt(d): what ATTN_LONG takes with them scaled.
bool attn_wants_scaled(int tokens, int heads, int d, int slots);
drf_status launch_attn_bf16(const AttnArgs& a, hipStream_t st);
drf_status launch_attn_long_bf16(const AttnArgs& a, hipStream_t st);
drf_status launch_attn_short_bf16(const AttnArgs& a, int queries, hipStream_t st);
int attn_short_items_at_once(int Nk, int d);    // work items of 32 queries that the chip holds of ATTN_SHORT
drf_status launch_attn_f32(const AttnArgs& a, hipStream_t st);

// The row-local part of a bf16 block as one launch (block_chain.hip): from the attention output, rows of the stream resid become
// x = resid + gate1 (proj(attn)), x += gate2 fc2(gelu(fc1(LN(x)))), stored over resid, then the next block's q | k | v of LN(x).
struct ChainArgs {
    const bf16_t* attn;             // [M][D]: the attention output, or NULL
    const bf16_t* kv_in;            // keys and values that the self-attention is computed from in the launch itself (heads of 64), with the queries
                                    // at q, or NULL; with neither, only the last part runs, of resid as it is or of the shares at part_in
    float* resid;                   // [M][D]
    const bf16_t* weights;          // packed units in the order of their use (launch_chain_pack): proj, (fc1, fc2) of every D hidden units, q, k, v
    const float *b_proj, *b_fc1, *b_fc2, *b_qkv;
    const float* mod;               // slot 0's gate1 | shift2 | scale2 | gate2 | next shift1 | next scale1, D each (the first four not read for the last part alone)
    int mod_ld, tokens, slots, mlp_ratio;
    bf16_t* qkv;                    // head-major planes of `plane` elements as EPI_STORE_HEADS writes them, or NULL
    // The form that the next launch computes its self-attention from; neither this nor qkv: no last part.  Keys, then values, of every slot and
    // head in groups of 32 keys of 64, as operand fragments: the first 16-byte piece of lane (l, quarter) in fragment (b, s) of the
    // keys is columns 32 s + 8 quarter .. + 7 of key 8 (l / 4) + l % 4 + 4 b, in fragment d of the values column 16 d + l of keys
    // 8 quarter .. + 7.  Other memory than kv_in.  The queries go to q (a workgroup reads and writes its own rows).
    bf16_t *q, *kv_out;
    size_t plane; int heads, hd; uint32_t hd_magic; int hd_shift; float q_scale;
    // For few rows (16 a workgroup) a block runs as two launches of several workgroups a row tile: the first deals the hidden units over
    // `parts`, each leaving its share of the stream at part_out[part][M][D]; the second adds the n_in shares at part_in up, stores the
    // stream, and deals q, k and v over `parts` (1: neither); with no q, k, v to follow it only adds and stores.
    int parts, n_in;
    float* part_out; const float* part_in;
};
bool chain_width(int D, int mlp_ratio);             // hidden sizes and ratios that have the kernel
// How a pass uses it: rows a workgroup takes (0: the block's launches one by one are faster), whether with the self-attention, which
// then wants its queries scaled by chain_q_scale(), and in how many parts of the hidden units and of q, k, v (1: in one launch).
struct ChainRoute { int rows; bool attention; int parts, qkv_parts; };
ChainRoute chain_route(int slots, int D, int mlp_ratio, int tokens, int hd);
float chain_q_scale();
// One D x D unit, rows n of w[n][0 .. D) at stride ld, into the kernel's layout.
drf_status launch_chain_pack(const bf16_t* w, int ld, int D, bf16_t* out, hipStream_t st);
drf_status launch_block_chain(const ChainArgs& a, int D, int rows, hipStream_t st);

struct DitDims { int D, P, T, gh, gw, C, H, W, patch, heads, d, R, L; };

// c = MLP(femb(tau)) + cond embedding; writes SiLU(c) as float [slots][D] and, if act_bf16 != NULL, bf16.
struct CondArgs {
    const float *t_w1, *t_b1, *t_w2, *t_b2, *c_w, *c_b, *table;
    const void* cond; int cond_kind, cond_dim;
    int D, slots;
    SlotMap map;
    float* act_f32; bf16_t* act_bf16;
    float* scratch;          // slots * (256 + 3 D) floats
};
drf_status launch_cond_embed(const CondArgs& a, hipStream_t st);

drf_status launch_patch_embed(const float* x, const SlotMap& map, const float* w, const float* b, const float* pos,
                              const DitDims& dm, int slots, float* resid, hipStream_t st);
// out = LN(resid) * (1 + scale) + shift (shift == NULL: plain LN); mod rows are per slot.
// add != NULL (bf16 [M][D], and add2 likewise if also != NULL): the rows normalised are x = (resid + add) + add2;
// write_back stores x over resid, otherwise resid is left as it was and the caller passes the same `add`
// again (with the next branch output as add2) to the launch that does write back.
drf_status launch_ln_modulate(float* resid, const bf16_t* add, const bf16_t* add2, bool write_back, const float* shift,
                              const float* scale, int mod_ld, int rows_per_slot, int M, int D, void* out, int out_f32,
                              hipStream_t st);
// The same with the output of a split GEMM as the last branch: x = (resid + add) + bf16(gate * (sum of the
// partials + bias)), stored over resid; add may be NULL.  Only for the widths that ln_partial_width accepts; out is bf16.
bool ln_partial_width(int D);
struct PartialBranch { PartialSum sum; const float *bias, *gate; };
drf_status launch_ln_modulate_partial(float* resid, const bf16_t* add, const PartialBranch& br, const float* shift, const float* scale,
                                      int mod_ld, int rows_per_slot, int M, int D, bf16_t* out, hipStream_t st);
drf_status launch_final(const float* resid, const float* shift, const float* scale, int mod_ld, const float* w,
                        const float* b, const DitDims& dm, int slots, float* eps_out, hipStream_t st);
drf_status launch_f32_to_bf16(const float* in, bf16_t* out, size_t n, hipStream_t st);

}  // namespace drf
