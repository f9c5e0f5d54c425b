// The prompt's forward as matrix-matrix products ("given input x", paper Sec. II-A; the target forward that fills the
// cache before the first speculative step).  A prompt of hundreds of rows is bound by the matrix cores, not by the HBM
// read of the weights, so it does not go through the weight-streaming kernel 16 rows at a time (which re-reads every
// weight per 16 rows) but through a tiled GEMM per projection whose weights leave HBM once per panel of up to 512 rows
// (the workgroups that share a weight tile sit on one XCD and find it in that XCD's L2).  The same GEMM with a plain
// epilogue (PF_PLAIN) serves the products of the FIT pass (sdfp_fit.hip.h).
//
// What it must preserve: the cache rows and the residual stream it produces are the ones the decode kernels would
// produce, bit for bit (a rolled-back cache equals a freshly prefilled one; row i of a prompt equals the one-row decode
// of the same prefix).  So every output is computed with the arithmetic of sdfp_stream.hip.h:
//   * the reduction dimension is cut into NSHARE = 8 interleaved shares (share p owns the 4 consecutive 64-byte steps
//     4p .. 4p+3 of every 2 KB block of a weight row); a share's partial sum is one chain of
//     v_mfma_f32_16x16x32_bf16 accumulations over its steps in ascending order, three per step (the three bfloat16
//     pieces of the float32 activation, in order), weights as the A operand, activations as the B operand;
//   * the output is ((((0 + P0) + P1) + ...) + P7) in float32;
//   * norm scale, rotary embedding, SwiGLU, residual add, bfloat16 rounding of keys / values, the sum of squares of a
//     row and the split of an activation into pieces use the shared helpers of sdfp_common.hip.h, built from single
//     float32 operations that the compiler cannot contract with their neighbours;
//   * attention runs the decode kernels' own attn_split on 16-row chunks, or its operations on the matrix cores
//     (k_pf_attn_mx).
// The GEMM therefore walks the reduction dimension share by share (a permutation of the usual order), which costs
// nothing: every step of it is still a whole 64-byte line of 16 weight rows.
//
// Layout of a panel of P prompt rows in the workspace: h [P][d] float32 residual stream (updated in place); xs, the
// three bfloat16 pieces of the current projection input, each piece in OPERAND ORDER (pf_xs_off): the B operand of one
// matrix-core step -- 16 rows x 64 bytes -- is one contiguous kilobyte, lane l's 16 bytes at l * 16, so that the GEMM
// stages a slab with contiguous reads and writes it to LDS as it comes; q, att [P][H*hd] float32; rs [P] float32.
#pragma once
#include <type_traits>
#include "sdfp_attn.hip.h"
#include "sdfp_prefill_plan.h"

namespace sdfp {

constexpr int PF_NSHARE = 8;             // shares of the reduction dimension (= waves of the decode kernels)
constexpr int PF_STEP_BYTES = 64;        // bytes of a weight row per matrix-core step (32 bfloat16)
constexpr int PF_SPS = 4;                // consecutive steps of a share per block
constexpr int PF_BLOCK_BYTES = PF_NSHARE * PF_SPS * PF_STEP_BYTES;   // 2 KB
constexpr int PF_TM = 64;                // prompt rows per workgroup tile
constexpr int PF_FRAG_BYTES = 16 * PF_STEP_BYTES;          // one B operand: a step of 16 prompt rows, lane l's 16 bytes at l * 16
constexpr int PF_SLAB_BYTES = 3 * (PF_TM / 16) * PF_SPS * PF_FRAG_BYTES;   // pieces x column tiles x steps: 48 KB
constexpr int PF_SLABS = 3;                                // slabs of LDS: one is multiplied, two are on their way
constexpr int PF_LDS_BYTES = PF_SLABS * PF_SLAB_BYTES;

// Byte offset, inside one piece of an input with rows of Kd values, of the 16-byte unit that holds values 8 * k8 .. + 7 of
// row m: [16-row tile][64-byte step][quarter of the step][row of the tile][16 bytes].  A piece spans a whole number of
// tiles: ceil(rows / 16) * 16 * Kd values.
__host__ __device__ __forceinline__ size_t pf_xs_off(int m, int k8, int Kd) {
    return ((size_t)(m >> 4) * (size_t)(Kd >> 5) + (size_t)(k8 >> 2)) * PF_FRAG_BYTES + (size_t)((k8 & 3) * 256 + (m & 15) * 16);
}
__host__ __device__ __forceinline__ size_t pf_xs_piece(int rows, int Kd) { return (size_t)((rows + 15) / 16 * 16) * (size_t)Kd; }

enum { PF_QKV = 0, PF_OPROJ = 1, PF_GATEUP = 2, PF_DOWN = 3, PF_PLAIN = 4 };   // PF_PLAIN: out = (base +) x W^T, nothing fused

struct PfGemm {
    const bf16_t* w[3];      // QKV: wq wk wv; gate/up: w_gate w_up; else the matrix in w[0]; row-major [N][Kd]
    const bf16_t* wt;        // the projection's matrices once more in tile order (pf_tile_weights), or nullptr
    const bf16_t* xs;        // the three pieces of the input rows, each in operand order (pf_xs_off)
    size_t xs_piece;         // elements between pieces (pf_xs_piece)
    int Kd;                  // reduction length
    int n_tiles;             // 16-row weight tiles of the projection
    int M;                   // valid prompt rows of the panel
    int pos0;                // absolute position of the panel's row 0
    const float* rs;         // [P] reciprocal RMS of the input rows (QKV, gate/up), else nullptr
    float* h;                // O / down: residual stream [P][d], updated in place
    float* q;                // QKV: queries [P][H*hd]
    bf16_t *kc, *vc;         // QKV: this layer's key / value planes [Hkv][max_seq][hd]
    bf16_t* xs_out;          // gate/up: the pieces of the feed-forward activation (rows of F values), in operand order
    size_t xs_out_piece;
    const float *cosT, *sinT;
    float* out;              // PF_PLAIN: [M][ldo] float32 result
    int ldo;                 // PF_PLAIN: elements between rows of out
    const float* base;       // PF_PLAIN: [M][ldo] float32 added to the product (may be out), or nullptr
    float* part;             // a projection dealt by shares: [8][P][part_ld] partial sums
    size_t part_arr;         // floats per array of part (P * part_ld)
    int part_ld;             // floats per row of part: the projection's outputs (16 * n_tiles)
    int n_nt;                // groups of 8 * NT weight tiles
    int my;                  // row tiles of the panel (64 rows each)
    int n_groups;            // workgroups that share a tile's reduction dimension: 1, 2, 4 or 8
    LayerDims L;
};

// ---- RMSNorm prologue of a projection, in two kernels.  k_pf_rownorm: the reciprocal RMS of every row from its sum of
// squares in the decode kernels' order -- one workgroup of 512 threads per prompt row; threads 0..447 are the decode
// kernels' staging threads: thread t adds the 8-value chunks t, t + 448, ... in ascending order, lanes are folded by
// the DPP tree, the eight wave sums are added in wave order (the last wave's is 0).  k_pf_split: the rows (times the
// gain, if any) split into pieces, written in operand order. ----------------------------------------------------------
__global__ __launch_bounds__(512) void k_pf_rownorm(const float* __restrict__ h, int d, float eps, float* __restrict__ rs) {
    __shared__ float ss[NWAVE];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* row = h + (size_t)m * d;
    const int nchunk = d >> 3;
    float s = 0.f;
    for (int c = tid; c < nchunk && wave != NWAVE - 1; c += WG_THREADS - 64) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(row + c * 8), b = *reinterpret_cast<const f32x4*>(row + c * 8 + 4);
        s = add_rn(s, sq8(a, b));
    }
    s = wave_sum_last(s);
    if (lane == 63) ss[wave] = s;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) t = add_rn(t, ss[w]);
        rs[m] = rms_recip(t, d, eps);
    }
}

// x [rows][Kd] float32 (times gain [Kd], or gain == nullptr) -> three pieces in operand order.  A wave takes a
// fragment -- a 64-byte step of a 16-row tile -- at a time: lane l reads the 8 values (l / 16) * 8 .. of the step of row
// l % 16 and writes its 16 bytes of each piece at l * 16 of the fragment, a contiguous kilobyte per piece.  Rows past
// the last one repeat it (a piece spans whole tiles; what those rows produce is never used).
__global__ __launch_bounds__(256) void k_pf_split(const float* __restrict__ x, const float* __restrict__ gain, int rows, int Kd,
                                                  bf16_t* __restrict__ xs, size_t xs_piece) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, gq = lane >> 4;
    const int S = Kd >> 5, n_frag = ((rows + 15) >> 4) * S;
    for (int f = blockIdx.x * 4 + (threadIdx.x >> 6); f < n_frag; f += gridDim.x * 4) {
        const int t = f / S, st = f - t * S;
        const int m = min(t * 16 + r16, rows - 1), k0 = st * 32 + gq * 8;
        const float* src = x + (size_t)m * Kd + k0;
        const f32x4 a = *reinterpret_cast<const f32x4*>(src), b = *reinterpret_cast<const f32x4*>(src + 4);
        float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        if (gain != nullptr) {
            const f32x4 g0 = *reinterpret_cast<const f32x4*>(gain + k0), g1 = *reinterpret_cast<const f32x4*>(gain + k0 + 4);
            v[0] = mul_rn(v[0], g0.x); v[1] = mul_rn(v[1], g0.y); v[2] = mul_rn(v[2], g0.z); v[3] = mul_rn(v[3], g0.w);
            v[4] = mul_rn(v[4], g1.x); v[5] = mul_rn(v[5], g1.y); v[6] = mul_rn(v[6], g1.z); v[7] = mul_rn(v[7], g1.w);
        }
        u32x4 piece[3];
        split3_bf16(v, piece);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(xs + p * xs_piece) + (size_t)f * PF_FRAG_BYTES + lane * 16) = piece[p];
    }
}

// The three kernels that stand between two projections, in one: the residual update of a projection dealt by shares
// (h += ((((0 + P0) + P1) + ...) + P7), k_pf_residual; left out when part == nullptr), the reciprocal RMS of the new row
// (k_pf_rownorm: same threads, same chunks, same order) and the pieces of the row times the gain in operand order
// (k_pf_split).  One workgroup per prompt row; a thread keeps its chunks of the row in registers between the steps
// (rows of at most PF_FUSED_MAX_D values).  The rows that pad the last 16-row tile are left as they are, as the gate/up
// GEMM leaves them in the pieces it writes: an operand column feeds its own output column only, and those are dropped.
constexpr int PF_FUSED_CHUNKS = 3;                                   // 8-value chunks a thread may hold
constexpr int PF_FUSED_MAX_D = PF_FUSED_CHUNKS * 8 * (WG_THREADS - 64);
__global__ __launch_bounds__(512) void k_pf_residual_norm_split(float* __restrict__ h, const float* __restrict__ part, size_t part_arr,
                                                                int d, float eps, const float* __restrict__ gain,
                                                                float* __restrict__ rs, bf16_t* __restrict__ xs, size_t xs_piece) {
    __shared__ float ss[NWAVE];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float* row = h + (size_t)m * d;
    const int nchunk = d >> 3;
    float v[PF_FUSED_CHUNKS][8];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < PF_FUSED_CHUNKS; ++i) {
        const int c = tid + i * (WG_THREADS - 64);
        if (c < nchunk && wave != NWAVE - 1) {
            f32x4 a = *reinterpret_cast<const f32x4*>(row + c * 8), b = *reinterpret_cast<const f32x4*>(row + c * 8 + 4);
            if (part != nullptr) {
                f32x4 ta = f32x4{0.f, 0.f, 0.f, 0.f}, tb = ta;
#pragma unroll
                for (int p = 0; p < PF_NSHARE; ++p) {
                    const float* src = part + (size_t)p * part_arr + (size_t)m * d + c * 8;
                    const f32x4 pa = *reinterpret_cast<const f32x4*>(src), pb = *reinterpret_cast<const f32x4*>(src + 4);
                    ta = f32x4{add_rn(ta.x, pa.x), add_rn(ta.y, pa.y), add_rn(ta.z, pa.z), add_rn(ta.w, pa.w)};
                    tb = f32x4{add_rn(tb.x, pb.x), add_rn(tb.y, pb.y), add_rn(tb.z, pb.z), add_rn(tb.w, pb.w)};
                }
                a = f32x4{add_rn(a.x, ta.x), add_rn(a.y, ta.y), add_rn(a.z, ta.z), add_rn(a.w, ta.w)};
                b = f32x4{add_rn(b.x, tb.x), add_rn(b.y, tb.y), add_rn(b.z, tb.z), add_rn(b.w, tb.w)};
                *reinterpret_cast<f32x4*>(row + c * 8) = a; *reinterpret_cast<f32x4*>(row + c * 8 + 4) = b;
            }
            s = add_rn(s, sq8(a, b));
            v[i][0] = a.x; v[i][1] = a.y; v[i][2] = a.z; v[i][3] = a.w; v[i][4] = b.x; v[i][5] = b.y; v[i][6] = b.z; v[i][7] = b.w;
        }
    }
    s = wave_sum_last(s);
    if (lane == 63) ss[wave] = s;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) t = add_rn(t, ss[w]);
        rs[m] = rms_recip(t, d, eps);
    }
    const int S = d >> 5;                                            // 64-byte steps of a row of pieces
#pragma unroll
    for (int i = 0; i < PF_FUSED_CHUNKS; ++i) {
        const int c = tid + i * (WG_THREADS - 64);
        if (c < nchunk && wave != NWAVE - 1) {
            const f32x4 g0 = *reinterpret_cast<const f32x4*>(gain + c * 8), g1 = *reinterpret_cast<const f32x4*>(gain + c * 8 + 4);
            const float x[8] = {mul_rn(v[i][0], g0.x), mul_rn(v[i][1], g0.y), mul_rn(v[i][2], g0.z), mul_rn(v[i][3], g0.w),
                                mul_rn(v[i][4], g1.x), mul_rn(v[i][5], g1.y), mul_rn(v[i][6], g1.z), mul_rn(v[i][7], g1.w)};
            u32x4 piece[3];
            split3_bf16(x, piece);
            // chunk c = step c / 4, bytes (c % 4) * 16 .. of it: lane slot (c % 4) * 16 + row % 16 of the fragment
            const size_t at = ((size_t)(m >> 4) * S + (c >> 2)) * PF_FRAG_BYTES + (size_t)(((c & 3) << 4) + (m & 15)) * 16;
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(xs + p * xs_piece) + at) = piece[p];
        }
    }
}

// embedding rows of a panel: h[m][:] = tok_emb[prompt[m]][:]
__global__ __launch_bounds__(256) void k_pf_embed(const int* __restrict__ prompt, const bf16_t* __restrict__ emb, int d, int V,
                                                  float* __restrict__ h) {
    const int m = blockIdx.x;
    const int tok = min(max(prompt[m], 0), V - 1);
    for (int k = threadIdx.x * 4; k < d; k += blockDim.x * 4) {
        const u32x2 r = *reinterpret_cast<const u32x2*>(emb + (size_t)tok * d + k);
        *reinterpret_cast<f32x4*>(h + (size_t)m * d + k) =
            f32x4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16),
                  __uint_as_float(r.y & 0xFFFF0000u)};
    }
}

// This lane's row (r16 = lane % 16) of weight tile t of a projection, in the caller's row-major matrices.
template <int KIND>
__device__ __forceinline__ const char* pf_weight_row(const PfGemm& a, int t, int r16) {
    const size_t pitch = (size_t)a.Kd * 2;
    const bool hi = r16 >= 8;
    if (KIND == PF_QKV) {          // tile = 8 rotary pairs of one head of wq, wk or wv: rows (i, i + hd / 2)
        const int hd = a.L.hd, H = a.L.H, Hkv = a.L.Hkv, tph = hd >> 4;
        const int hs = t / tph, jj = t - hs * tph;
        const int sel = hs < H ? 0 : (hs < H + Hkv ? 1 : 2);
        const int head = hs - (sel == 0 ? 0 : (sel == 1 ? H : H + Hkv));
        const int row = head * hd + jj * 8 + (r16 & 7) + (hi ? (hd >> 1) : 0);
        return (const char*)a.w[sel] + (size_t)row * pitch;
    }
    if (KIND == PF_GATEUP)         // tile = 8 gate rows and the 8 up rows of the same units
        return (const char*)a.w[hi ? 1 : 0] + (size_t)(t * 8 + (r16 & 7)) * pitch;
    return (const char*)a.w[0] + (size_t)(t * 16 + r16) * pitch;
}

// The matrices of a projection once more, in tile order: tile t, step s -> one kilobyte, lane l's 16 bytes of the A
// operand (row l % 16 of the tile, bytes (l / 16) * 16 .. of the step) at l * 16.  The GEMM then reads a step of a tile
// as one contiguous kilobyte.  Read row by row the same step is 64 separate 16-byte accesses of the first-level cache
// (adjacent lanes hold different rows), which that cache serves at about one per cycle: measured on resident data,
// 9.6 TB/s against 32 TB/s for contiguous kilobytes -- enough for a kernel bound by HBM, not for one whose weights come
// from the L2 cache eight times over.  a: w, Kd, n_tiles, L as for the GEMM.
template <int KIND>
__global__ __launch_bounds__(256) void k_pf_tile_weights(PfGemm a, bf16_t* __restrict__ dst) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, gq = lane >> 4;
    const int S = a.Kd * 2 / PF_STEP_BYTES;
    const size_t n_frag = (size_t)a.n_tiles * S;
    for (size_t f = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); f < n_frag; f += (size_t)gridDim.x * 4) {
        const int t = (int)(f / S), s = (int)(f - (size_t)t * S);
        const char* src = pf_weight_row<KIND>(a, t, r16) + s * PF_STEP_BYTES + gq * 16;
        *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(dst) + f * PF_FRAG_BYTES + lane * 16) =
            *reinterpret_cast<const u32x4*>(src);
    }
}

// ---- the GEMM.  A workgroup computes 8 / WJ * NT weight tiles x PF_TM prompt rows; WJ waves share NT weight tiles, each
// with its part of the four 16-row column tiles, so that an input piece read from LDS feeds NT matrix-core instructions:
// WJ = 1 with three or four tiles (a weight is read by one wave only), 2 where a workgroup has 8 or 16 tiles (with one or two
// tiles per wave and all columns the LDS reads took as long as the matrix cores or longer).  Weights go from memory straight
// into the A operand (lane l: row l % 16, bytes (l / 16) * 16 .. of the step, as in the decode kernels), WD slabs ahead; the
// input pieces of a slab -- the 4 steps that one share owns in one block, for all 64 prompt rows -- are staged in LDS, two
// slabs ahead in three buffers, and read as the B operand (lane l: prompt row l % 16, the same bytes of the step).
// What bounds it: large tiles the matrix cores at the power limit (7B gate/up, 512 rows: 224 us, 1.24 PFLOP/s counting the
// three passes; hipBLASLt's bf16 product of that size 286 us), 16 tiles 337 -> 318 us with this pipeline (Llama-3-8B gate/up),
// 8 tiles the read of the weights (7B gate/up at 37 rows 65 -> 57 us, 3.2 TB/s).
//
// Workgroups that read the same weights (the panel's row tiles of one weight tile group) are neighbours on one XCD,
// so the weights come from HBM once and from that XCD's L2 afterwards: workgroup id -> XCD id % 8, place id / 8 on it;
// a place is (column c = (tile group, share group), row tile), row tile fastest; column c lives on XCD c % 8.
//
// PARTIAL: the projection is too narrow to fill the chip with whole outputs (O and down projections; QKV of a short
// prompt), so the shares of the reduction dimension are dealt to n_groups workgroups per tile; each writes its shares'
// partial sums P_p to part[p][row][N], and k_pf_residual (k_pf_finish_qkv) adds them in share order.
// JT: 16-row column tiles of the workgroup tile that are multiplied (4; 1 or 2 for a panel of at most 16 or 32 rows,
// which then costs a quarter or half of the matrix-core instructions and LDS reads, and fetches as much less).
template <int KIND, int NT, bool PARTIAL, int JT = 4, int WJ = 1>
__global__ __launch_bounds__(WG_THREADS, 1) void k_pf_gemm(PfGemm a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, gq = lane >> 4;
    const int xcd = blockIdx.x & 7, place = blockIdx.x >> 3;
    const int col = (place / a.my) * 8 + xcd;
    if (col >= a.n_nt * a.n_groups) return;                 // uniform over the workgroup
    const int grp = col % a.n_groups;
    const int m0 = (place % a.my) * PF_TM;                  // first prompt row of the workgroup tile
    constexpr int JW = JT / WJ;                             // the wave's column tiles, j0 ..
    const int j0 = (wave % WJ) * JW;
    const int t0 = (col / a.n_groups) * (8 / WJ * NT) + wave / WJ * NT;   // the wave's first weight tile
    const int pitch = a.Kd * 2;                             // bytes per weight row
    const int S = pitch / PF_STEP_BYTES;                    // steps per weight row
    const int nblk = (S + PF_NSHARE * PF_SPS - 1) / (PF_NSHARE * PF_SPS);
    const int hd = a.L.hd, H = a.L.H, Hkv = a.L.Hkv, half = hd >> 1, tph = hd >> 4;

    // This lane's 16 bytes of step 0 of tile t (tiles past the end repeat the last one; their outputs are dropped), and
    // the bytes from one step to the next: in the tiled copy a step of a tile is a kilobyte, in the caller's matrices
    // 64 bytes of each of the tile's rows.
    const bool tiled = a.wt != nullptr;
    const int wstep = tiled ? PF_FRAG_BYTES : PF_STEP_BYTES;
    const char* wrow[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tc = min(t0 + t, a.n_tiles - 1);
        wrow[t] = tiled ? (const char*)a.wt + (size_t)tc * S * PF_FRAG_BYTES + lane * 16
                        : pf_weight_row<KIND>(a, tc, r16) + gq * 16;
    }

    // Staging of a slab: 3 pieces x 64 prompt rows x 256 bytes = 48 fragments of 1 KB, 6 per wave.  The slab lies in LDS
    // as it lies in memory, in operand order: fragment f = (piece * 4 + column tile) * 4 + step, lane l's 16 bytes
    // (prompt row l % 16 of the column tile, bytes (l / 16) * 16 .. of the step) at l * 16 -- a wave reads a B operand
    // as one contiguous kilobyte, free of bank conflicts however the hardware groups the lanes, and a fragment travels
    // from memory to LDS with one load-to-LDS instruction per wave (lane l's 16 bytes land at l * 16), through no
    // register.
    const char* xs_base = (const char*)a.xs;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    // slab i of the walk: share p = i / nblk, block b = i % nblk; its first byte in a row, and how many of its 4 steps exist
    auto slab_byte0 = [&](int i) { return (i % nblk) * PF_BLOCK_BYTES + (i / nblk) * (PF_SPS * PF_STEP_BYTES); };
    auto slab_steps = [&](int i) { return max(0, min(PF_SPS, S - ((i % nblk) * (PF_NSHARE * PF_SPS) + (i / nblk) * PF_SPS))); };
    const int spg = PF_NSHARE / a.n_groups;                 // shares per group
    const int i_lo = grp * spg * nblk, i_hi = i_lo + spg * nblk;

    f32x4 total[PARTIAL ? 1 : NT][PARTIAL ? 1 : JW], acc[NT][JW];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < JW; ++j) {
            acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (!PARTIAL) total[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

    // Every load of the loop below is unconditional and its address clamped into the row: a load under a condition makes
    // the compiler wait, at the join, for everything in flight, and the pipeline (pieces one or two slabs ahead, weights up to
    // three) would stall once per step.  What a clamped load brings is never used: the steps a slab does not have are skipped.
    // the wave's weight steps, WD slabs of them: a step's registers take the step WD slabs further on when it is multiplied
    constexpr int WD = pf_weight_depth(NT);
    // Large tiles (three or four per wave and all columns: bound by the matrix cores) fetch the pieces one slab ahead, behind the
    // slab's first step: the deeper pipeline of the others is 0.7 % slower there.
    constexpr bool ONE_AHEAD = pf_one_ahead(NT, WJ);
    u32x4 wa[WD][NT][PF_SPS];
    const int last_tile16 = (a.M - 1) >> 4;
    // Slab i into LDS buffer buf; wave w fetches fragments w, w + 8, ...  The loads are counted with the wave's other
    // vector memory loads and complete in order with them.  They are issued from an asm statement: told what they are,
    // the compiler makes every later LDS read that it cannot prove disjoint (the other buffer) wait for them, i.e. for
    // all memory traffic of the wave, once per slab.  So the kernel waits for them itself, before the barrier that lets
    // anybody read the buffer; the compiler's own waits for the weight loads merely count up to 6 loads too few in
    // flight, which makes them wait for a little more than they need, never less.
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds;
    auto fetch_slab = [&](int i, int buf) {
        const int byte0 = slab_byte0(i);
#pragma unroll
        for (int u = 0; u < 6; ++u) {
            const int frag = wave_u + u * NWAVE, piece = frag >> 4;
            if (!pf_fetched(JT, frag)) continue;   // a column tile that is not multiplied (wave-uniform)
            const int tile16 = min((m0 >> 4) + ((frag >> 2) & 3), last_tile16);
            const int step = min((byte0 >> 6) + (frag & 3), S - 1);
            const char* src = xs_base + (size_t)piece * a.xs_piece * 2 + ((size_t)tile16 * S + step) * PF_FRAG_BYTES + lane * 16;
            // M0 = LDS byte address of the fragment (wave-uniform); lane l's 16 bytes land at M0 + l * 16
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                         :
                         : "s"(lds0 + (unsigned)(buf * PF_SLAB_BYTES + frag * PF_FRAG_BYTES)), "v"(src)
                         : "memory");   // (M0 is not allocatable: the compiler sets it in front of each of its own uses)
        }
    };
    auto load_weight_step = [&](int byte0, int s, u32x4 (&w)[NT][PF_SPS]) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
            w[t][s] = *reinterpret_cast<const u32x4*>(wrow[t] + (size_t)(min((byte0 >> 6) + s, S - 1) * wstep));
    };
    const int i_last = i_hi - 1;                               // past the end the last slab is fetched again, unused
    fetch_slab(i_lo, 0);
#pragma unroll
    for (int s = 0; s < PF_SPS; ++s) load_weight_step(slab_byte0(i_lo), s, wa[0]);
    if (!ONE_AHEAD) fetch_slab(min(i_lo + 1, i_last), 1);
#pragma unroll
    for (int w = 1; w < WD; ++w)
#pragma unroll
        for (int s = 0; s < PF_SPS; ++s) load_weight_step(slab_byte0(min(i_lo + w, i_last)), s, wa[w]);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(pf_wait_first(NT, JT, WJ)) : "memory");
    __syncthreads();
    int buf = 0;                                               // LDS slab of slab i
    // tail: the walk's last slabs, behind whole rounds of WD; their pieces and weights are on their way or here, there is
    // nothing more to request.
    auto slab = [&](int i, u32x4 (&w)[NT][PF_SPS], auto tail) {
        constexpr bool TAIL = decltype(tail)::value;
        const int nst = slab_steps(i);
        const int byte0_next = slab_byte0(min(i + WD, i_last));
        // The pieces of the slab after the next one, into the buffer whose last readers passed the barrier in front of this
        // slab.  Two slabs ahead and in front of this slab's weight loads: memory answers in order, so the wait for the next
        // slab's pieces at the end of this slab is for nothing younger than the previous slab's start.
        if (!ONE_AHEAD && !TAIL) fetch_slab(min(i + 2, i_last), buf == 0 ? 2 : buf - 1);
        const char* xb = lds + buf * PF_SLAB_BYTES + j0 * (PF_SPS * PF_FRAG_BYTES) + lane * 16;
        auto frag = [&](int s, int j, int p) {
            return *reinterpret_cast<const u32x4*>(xb + ((p * 4 + j) * PF_SPS + s) * PF_FRAG_BYTES);
        };
        // every accumulator sees its three pieces in order; neighbours in the instruction stream are independent
        auto multiply = [&](int s, int j, const u32x4 (&x3)[3]) {
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, w[t][s]), __builtin_bit_cast(bf16x8, x3[p]), acc[t][j], 0, 0, 0);
        };
        // Straight-line code for every slab: the B operands of a (step, column tile) are read from LDS while the previous
        // one is multiplied (read and used back to back, their latency showed in every group of instructions).  A step
        // that the slab does not have (the ragged end of a row) is multiplied with weights of zero: it adds +-0 to sums
        // that started at +0, which changes no bit -- the decode kernels multiply such a step by a block of zeros.
        u32x4 cur[3], nxt[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) cur[p] = frag(0, 0, p);
#pragma unroll
        for (int s = 0; s < PF_SPS; ++s) {
            if (s >= nst) {   // uniform; rare
#pragma unroll
                for (int t = 0; t < NT; ++t) w[t][s] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int j = 0; j < JW; ++j) {
                const int g = s * JW + j + 1;
                if (g < JW * PF_SPS) {
#pragma unroll
                    for (int p = 0; p < 3; ++p) nxt[p] = frag(g / JW, g % JW, p);
                }
                __builtin_amdgcn_sched_barrier(0);   // the reads stay in front of the instructions that hide them
                multiply(s, j, cur);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < 3; ++p) cur[p] = nxt[p];
            }
            if (!TAIL) load_weight_step(byte0_next, s, w);           // this step's registers are free
            if (ONE_AHEAD && s == 0) fetch_slab(min(i + 1, i_last), buf ^ 1);
        }
        if ((i + 1) % nblk == 0) {   // the share's partial sums are complete
            const int p = i / nblk;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int j = 0; j < JW; ++j) {
                    if (PARTIAL) {
                        const int tile = t0 + t, m = m0 + (j0 + j) * 16 + r16;
                        if (tile < a.n_tiles && m < a.M)
                            *reinterpret_cast<f32x4*>(a.part + (size_t)p * a.part_arr + (size_t)m * a.part_ld + tile * 16 + gq * 4) = acc[t][j];
                    } else {     // added in share order
                        f32x4& T = total[PARTIAL ? 0 : t][PARTIAL ? 0 : j];
                        T.x = add_rn(T.x, acc[t][j].x); T.y = add_rn(T.y, acc[t][j].y);
                        T.z = add_rn(T.z, acc[t][j].z); T.w = add_rn(T.w, acc[t][j].w);
                    }
                    acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(TAIL ? 0 : pf_wait_slab(NT, JT, WJ)) : "memory");   // the next slab's pieces
        __syncthreads();
        buf = ONE_AHEAD ? buf ^ 1 : (buf == PF_SLABS - 1 ? 0 : buf + 1);
    };
    int i = i_lo;
    for (; i + WD <= i_hi; i += WD) {
#pragma unroll
        for (int w = 0; w < WD; ++w) slab(i + w, wa[w], std::false_type{});
    }
#pragma unroll
    for (int w = 0; w + 1 < WD; ++w)
        if (i + w < i_hi) slab(i + w, wa[w], std::true_type{});
    // Pieces fetched past the end have landed before the workgroup gives its LDS back.  And every weight load above has a use,
    // here: one that brings nothing that is multiplied could be dropped otherwise, and the waits count it.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (WD > 1) {
#pragma unroll
        for (int w = 0; w < WD; ++w)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int s = 0; s < PF_SPS; ++s) asm volatile("" ::"v"(wa[w][t][s]));
    }
    if (PARTIAL) return;

    // ---- epilogue.  Lane l holds, per tile, prompt row (column) l % 16 and output rows 4 * (l / 16) .. + 3 of the tile.
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tile = t0 + t;
        if (tile >= a.n_tiles) continue;
#pragma unroll
        for (int j = 0; j < JW; ++j) {
            const int m = m0 + (j0 + j) * 16 + r16;
            f32x4 v = total[PARTIAL ? 0 : t][PARTIAL ? 0 : j];
            if (KIND == PF_PLAIN) {
                if (m < a.M) {
                    float* o = a.out + (size_t)m * a.ldo + tile * 16 + gq * 4;
                    if (a.base != nullptr) {
                        const f32x4 r = *reinterpret_cast<const f32x4*>(a.base + (size_t)m * a.ldo + tile * 16 + gq * 4);
                        v = f32x4{add_rn(r.x, v.x), add_rn(r.y, v.y), add_rn(r.z, v.z), add_rn(r.w, v.w)};
                    }
                    *reinterpret_cast<f32x4*>(o) = v;
                }
                continue;
            }
            if (KIND == PF_OPROJ || KIND == PF_DOWN) {
                if (m < a.M) {
                    float* o = a.h + (size_t)m * a.L.d + tile * 16 + gq * 4;
                    const f32x4 r = *reinterpret_cast<const f32x4*>(o);
                    *reinterpret_cast<f32x4*>(o) = f32x4{add_rn(r.x, v.x), add_rn(r.y, v.y), add_rn(r.z, v.z), add_rn(r.w, v.w)};
                }
                continue;
            }
            // QKV, gate/up: rows r and r + 8 of the tile form a pair; they sit in lanes l and l + 32
            const float rsm = a.rs[min(m, a.M - 1)];
            v = f32x4{mul_rn(v.x, rsm), mul_rn(v.y, rsm), mul_rn(v.z, rsm), mul_rn(v.w, rsm)};
            f32x4 o2;
            o2.x = __shfl_xor(v.x, 32); o2.y = __shfl_xor(v.y, 32); o2.z = __shfl_xor(v.z, 32); o2.w = __shfl_xor(v.w, 32);
            if (gq >= 2 || m >= a.M) continue;          // lanes 0..31 hold rows 0..7 (first of each pair)
            float lo[4] = {v.x, v.y, v.z, v.w}, hi[4] = {o2.x, o2.y, o2.z, o2.w};
            if (KIND == PF_GATEUP) {
                const int u = tile * 8 + gq * 4;        // units u .. u + 3 of prompt row m
                float act[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) act[e] = swiglu(lo[e], hi[e]);
                // pieces of 4 consecutive values (the split works on 8; the upper 4 are zeros and are not stored)
                const float x8[8] = {act[0], act[1], act[2], act[3], 0.f, 0.f, 0.f, 0.f};
                u32x4 piece[3];
                split3_bf16(x8, piece);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(a.xs_out + p * a.xs_out_piece) +
                                              pf_xs_off(m, u >> 3, a.L.F) + (u & 4) * 2) = u32x2{piece[p].x, piece[p].y};
            } else {   // QKV
                const int hs = tile / tph, i0 = (tile - hs * tph) * 8 + gq * 4;   // dims i0 .. i0 + 3 and + half
                const int pos = a.pos0 + m;
                if (hs < H + Hkv) {
                    const f32x4 c = *reinterpret_cast<const f32x4*>(a.cosT + (size_t)pos * half + i0);
                    const f32x4 sn = *reinterpret_cast<const f32x4*>(a.sinT + (size_t)pos * half + i0);
                    rotary_pair(lo[0], hi[0], c.x, sn.x); rotary_pair(lo[1], hi[1], c.y, sn.y);
                    rotary_pair(lo[2], hi[2], c.z, sn.z); rotary_pair(lo[3], hi[3], c.w, sn.w);
                }
                if (hs < H) {
                    float* o = a.q + (size_t)m * H * hd + (size_t)hs * hd + i0;
                    *reinterpret_cast<f32x4*>(o) = f32x4{lo[0], lo[1], lo[2], lo[3]};
                    *reinterpret_cast<f32x4*>(o + half) = f32x4{hi[0], hi[1], hi[2], hi[3]};
                } else {
                    const bool isk = hs < H + Hkv;
                    const int kvh = isk ? hs - H : hs - H - Hkv;
                    bf16_t* o = (isk ? a.kc : a.vc) + ((size_t)kvh * a.L.max_seq + pos) * hd + i0;
                    *reinterpret_cast<u32x2*>(o) = u32x2{(unsigned)f32_to_bf16(lo[0]) | ((unsigned)f32_to_bf16(lo[1]) << 16),
                                                         (unsigned)f32_to_bf16(lo[2]) | ((unsigned)f32_to_bf16(lo[3]) << 16)};
                    *reinterpret_cast<u32x2*>(o + half) = u32x2{(unsigned)f32_to_bf16(hi[0]) | ((unsigned)f32_to_bf16(hi[1]) << 16),
                                                                (unsigned)f32_to_bf16(hi[2]) | ((unsigned)f32_to_bf16(hi[3]) << 16)};
                }
            }
        }
    }
}


// O / down projection in PARTIAL form: h = base + ((((0 + P0) + P1) + ...) + P7), 4 outputs per thread; base may be h, or
// nullptr for zero
__global__ __launch_bounds__(256) void k_pf_residual(const float* base, float* h, const float* __restrict__ part, size_t part_arr, int n4) {
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n4; c += gridDim.x * blockDim.x) {
        f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < PF_NSHARE; ++p) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(part + (size_t)p * part_arr + (size_t)c * 4);
            t = f32x4{add_rn(t.x, v.x), add_rn(t.y, v.y), add_rn(t.z, v.z), add_rn(t.w, v.w)};
        }
        const f32x4 r = base != nullptr ? *reinterpret_cast<const f32x4*>(base + (size_t)c * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4*>(h + (size_t)c * 4) = f32x4{add_rn(r.x, t.x), add_rn(r.y, t.y), add_rn(r.z, t.z), add_rn(r.w, t.w)};
    }
}

// ---- QKV dealt by shares (short prompts: a panel of a few dozen rows is bound by the read of the weights and needs
// more workgroups than the projection's 96 tile groups give): the GEMM leaves the 8 partial sums of every output in
// part, this kernel adds them in share order and runs the projection's epilogue -- the same operations as the GEMM's
// own. ------------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ float pf_share_sum(const float* part, size_t part_arr, size_t at) {
    float t = 0.f;
#pragma unroll
    for (int p = 0; p < PF_NSHARE; ++p) t = add_rn(t, part[(size_t)p * part_arr + at]);
    return t;
}
// one thread per (prompt row, tile, rotary pair): rows pr and pr + 8 of the tile
__global__ __launch_bounds__(256) void k_pf_finish_qkv(PfGemm a) {
    const int hd = a.L.hd, H = a.L.H, Hkv = a.L.Hkv, half = hd >> 1, tph = hd >> 4;
    const int n = a.M * a.n_tiles * 8;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += gridDim.x * blockDim.x) {
        const int pr = idx & 7, tile = (idx >> 3) % a.n_tiles, m = (idx >> 3) / a.n_tiles;
        const size_t at = (size_t)m * a.part_ld + tile * 16 + pr;
        const float rsm = a.rs[m];
        float lo = mul_rn(pf_share_sum(a.part, a.part_arr, at), rsm), hi = mul_rn(pf_share_sum(a.part, a.part_arr, at + 8), rsm);
        const int hs = tile / tph, i = (tile - hs * tph) * 8 + pr, pos = a.pos0 + m;
        if (hs < H + Hkv) rotary_pair(lo, hi, a.cosT[(size_t)pos * half + i], a.sinT[(size_t)pos * half + i]);
        if (hs < H) {
            float* o = a.q + (size_t)m * H * hd + (size_t)hs * hd + i;
            o[0] = lo; o[half] = hi;
        } else {
            const bool isk = hs < H + Hkv;
            const int kvh = isk ? hs - H : hs - H - Hkv;
            bf16_t* o = (isk ? a.kc : a.vc) + ((size_t)kvh * a.L.max_seq + pos) * hd + i;
            o[0] = f32_to_bf16(lo); o[half] = f32_to_bf16(hi);
        }
    }
}
// ---- attention of a panel: the decode kernels' attn_split on 16-row chunks.  A workgroup takes (chunk, KV head) items
// and runs the chunk's splits one after another into a region of its own (split partials), so that the last call merges
// them in ascending split order, the operations and the order of the forward kernel's merge (attn_merge).
struct PfAttn {
    const float* q;        // [P][H*hd] of the panel
    float* att;            // [P][H*hd]
    const bf16_t *kc, *vc; // this layer's planes
    float* part;           // per workgroup: part_o [n_splits][16][grp][hd] then part_ml [n_splits][16][grp][2]
    size_t part_stride;    // floats per workgroup region
    size_t part_ml_off;    // floats from a region's start to its part_ml
    int M;                 // valid rows of the panel
    int pos0;              // absolute position of the panel's row 0
    LayerDims L;
};
// LONGCTX: the panel ends beyond 8 attention splits (1024 positions); see attn_split (the instance for shorter prompts
// is 5 % faster without that code)
template <int LPP, bool LONGCTX>
__global__ __launch_bounds__(WG_THREADS, 4) void k_pf_attn(PfAttn a) {   // 4 waves per SIMD: two workgroups per compute unit (three: spills, slower)
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int grp = a.L.H / a.L.Hkv;
    const int n_chunks = (a.M + MAX_ROWS - 1) / MAX_ROWS;
    AttnArgs aa;
    aa.part_o = a.part + (size_t)blockIdx.x * a.part_stride;
    aa.part_ml = aa.part_o + a.part_ml_off;
    aa.part_H = grp;
    aa.L = a.L; aa.st = nullptr;
    for (int it = blockIdx.x; it < n_chunks * a.L.Hkv; it += gridDim.x) {
        const int c = it / a.L.Hkv, g = it - c * a.L.Hkv;
        aa.q = a.q + (size_t)c * MAX_ROWS * a.L.H * a.L.hd;
        aa.att = a.att + (size_t)c * MAX_ROWS * a.L.H * a.L.hd;
        aa.rows = Rows{min(MAX_ROWS, a.M - c * MAX_ROWS), ROWS_PROMPT, a.pos0 + c * MAX_ROWS};
        aa.part_h0 = g * grp;
        const int n_active = (aa.rows.off + aa.rows.M + ATT_SL - 1) / ATT_SL;
        for (int split = 0; split < n_active; ++split) {
            attn_split<bf16_t, LPP, 0, true, LONGCTX>(a.kc, a.vc, aa, reinterpret_cast<float*>(lds), split, g);
            __syncthreads();
        }
    }
}

// ---- the same attention on the float32 matrix cores (head_dim 64 and 128).  v_mfma_f32_16x16x4_f32 computes every output
// as a chain of four fused multiply-adds in ascending k, each correctly rounded (measured on 2 million products, wide
// exponents and denormals among them: no bit differs), so it can run attn_split's own operations:
//   scores   one instruction with C = 0 forms the 4-dim partial products of 16 keys x 16 queries; the tree of
//            group_sum_dpp over the hd / 4 partial products is plain register adds;
//   values   the chain of an output over a wave's positions, per position slot, is NL / 4 instructions; the slots' tree and
//            the sum over the decode kernels' waves, in their order, are plain register adds.
// A wave owns a tile of 16 prompt rows x one query head; the scores of a tile land on the lanes in the operand order of
// the value products (key rows of a tile are dealt to make it so), so probabilities never leave the registers and
// nothing crosses lanes but the soft-max statistics.
// What bounds it: per tile and split of 128 positions 512 instructions (head_dim 128) that hold a matrix core 32 cycles
// each, and 2700 vector instructions of 4.  Counters at 4096 positions: matrix cores 48 % busy, vector issue 38 %, the rest
// barriers and staging.  Measured against k_pf_attn on the vector ALUs: 8 KV heads x 4 queries, 512 rows at 3584-4096
// positions 1740 -> 475 us (the 4096-token prompt 429 -> 244 ms); 32 heads, 512 rows 122 -> 70 us.
//
// Positions.  attn_split walks position j = l * NC + ch, NC = 8 waves x PPL slots, chain ch = wave * PPL + slot over
// l = 0 .. NL - 1.  Here lane group gq = lane / 16 holds l = gq + 4 i, i < NI = NL / 4, of every chain: unit
// u = ch * NI + i (0..31) of group gq is position (gq + 4 i) * NC + ch.
//
// Workgroup: 4 tiles of one KV head (consecutive in (chunk, query head) order) x 2 splits at a time: waves 0-3 take the
// even splits, waves 4-7 the odd ones, each half stages its split's keys and values in LDS in operand order; the next
// pair is loaded into registers meanwhile.  Split partials go to a slot of scratch memory of the workgroup's own and are
// merged at the end, as attn_split does, by the same operations in ascending split order.
struct PfAttnMx {
    const float* q;        // [P][H*hd] of the panel
    float* att;            // [P][H*hd]
    const bf16_t *kc, *vc; // this layer's planes
    float* part;           // one slot per workgroup: [n_slots][64][hd] partials, then [n_slots][64][2] statistics
    size_t part_stride;    // floats per slot
    size_t part_ml_off;    // floats from a slot's start to its statistics
    int M, pos0;           // valid rows of the panel, absolute position of row 0
    LayerDims L;
};
constexpr int PFX_TILES = PF_MX_TILES;             // query tiles per workgroup
constexpr int PFX_QUERIES = PFX_TILES * 16;
static_assert(PF_CHUNK == MAX_ROWS && PF_SPLIT == ATT_SL, "the plan's cuts are the kernels'");
static_assert(PF_VALU_MAX_SPLITS * 8 <= attn_lds_bytes(16, 0, ATT_QC_PANEL, true) && PF_VALU_MAX_SPLITS * 8 <= attn_lds_bytes(32, 0, ATT_QC_PANEL, true) &&
              PF_VALU_MAX_SPLITS * 8 <= attn_lds_bytes(64, 0, ATT_QC_PANEL, true), "one query's statistics fit k_pf_attn's LDS");
__host__ __device__ constexpr size_t pfx_lds_bytes(int hd) { return (size_t)2 * 2 * ATT_SL * hd * 2; }   // 2 splits x (K, V)

__device__ __forceinline__ f32x4 add4_rn(const f32x4& a, const f32x4& b) {
    return f32x4{add_rn(a.x, b.x), add_rn(a.y, b.y), add_rn(a.z, b.z), add_rn(a.w, b.w)};
}
// value u (of 8 packed bfloat16) of an operand quad, widened
__device__ __forceinline__ float bf16_of8(const u32x4& r, int u) {
    const unsigned w = u < 2 ? r.x : (u < 4 ? r.y : (u < 6 ? r.z : r.w));
    return __uint_as_float((u & 1) ? (w & 0xFFFF0000u) : (w << 16));
}
// lower halves (hi = false) or upper halves of two words, a's first
__device__ __forceinline__ unsigned pack_halves(unsigned a, unsigned b, bool hi) {
    return __builtin_amdgcn_perm(b, a, hi ? 0x07060302u : 0x05040100u);
}
// x + y' where lanes 0-31 get x of their own and of lane + 32, lanes 32-63 y of both (and the same by 16-lane rows)
__device__ __forceinline__ float fold32(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return add_rn(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float fold16(float x, float y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return add_rn(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int LPP>
__global__ __launch_bounds__(WG_THREADS, 2) void k_pf_attn_mx(PfAttnMx a) {
    constexpr int HD = LPP * 4, PPL = 64 / LPP, NC = NWAVE * PPL, NL = ATT_SL / NC, NI = NL / 4;
    constexpr int GQ = HD / 32;            // 16-byte fragments per lane of a key tile (8 4-dim groups each)
    constexpr int DT = HD / 16;            // 16-dim tiles of the output
    constexpr int DQ = HD / 4;             // 4-dim quads of a value row
    constexpr int NU = HD / 64;            // staging units per thread, of keys and of values
    static_assert(NI >= 1 && NC * NI == 32 && NWAVE == 8 && ATT_SL == 128, "32 units per lane group");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, gq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tl = wave & 3, sp = wave >> 2, ht = tid & 255;
    const int H = a.L.H, Hkv = a.L.Hkv, grp = H / Hkv;
    const int n_chunks = (a.M + 15) >> 4, n_tk = n_chunks * grp, n_tg = (n_tk + PFX_TILES - 1) / PFX_TILES;
    const float scale = 1.0f / sqrtf((float)HD);
    char* const kb = lds + sp * (2 * ATT_SL * HD * 2);
    char* const vb = kb + ATT_SL * HD * 2;
    float* const slot = a.part + (size_t)blockIdx.x * a.part_stride;
    float* const slot_ml = slot + a.part_ml_off;
    auto pos_of = [](int u, int g) { return (g + 4 * (u % NI)) * NC + u / NI; };   // position in its split

    // items: KV head fastest (a head's workgroups share an XCD and its L2 where Hkv is a multiple of 8), longest rows first
    for (int it = blockIdx.x; it < n_tg * Hkv; it += gridDim.x) {
        const int g = it % Hkv, tg = n_tg - 1 - it / Hkv;
        auto chunk_end = [&](int c) { return a.pos0 + min(a.M, c * 16 + 16); };   // positions a chunk's attention covers
        const int t_last = min(tg * PFX_TILES + PFX_TILES, n_tk) - 1;
        const int end_wg = chunk_end(t_last / grp);
        const int n_act_wg = (end_wg + ATT_SL - 1) / ATT_SL;
        // this wave's tile (a tile past the last one does no work)
        const int t = tg * PFX_TILES + tl;
        const bool live = t < n_tk;
        const int c = min(t, n_tk - 1) / grp, hq = g * grp + min(t, n_tk - 1) % grp;
        const int end = chunk_end(c), rows = min(16, a.M - c * 16), n_act = (end + ATT_SL - 1) / ATT_SL;
        const int my_pos = a.pos0 + c * 16 + r16;          // absolute position of this lane's query row

        // the queries, operand B of the score products: lane (row r16, gq) holds dims 4 G + gq
        float qv[DQ];
        {
            const float* qrow = a.q + (size_t)(c * 16 + min(r16, rows - 1)) * H * HD + (size_t)hq * HD + gq;
#pragma unroll
            for (int G = 0; G < DQ; ++G) qv[G] = qrow[4 * G];
        }
        const char* kp = reinterpret_cast<const char*>(a.kc + (size_t)g * a.L.max_seq * HD);
        const char* vp = reinterpret_cast<const char*>(a.vc + (size_t)g * a.L.max_seq * HD);
        u32x4 kr[NU][4];
        u32x2 vr[NU][8];
        // loads are unconditional, addresses clamped to the last row; rows past it are replaced by zeros when they are staged
        auto fetch = [&](int split) {
            const int start = min(split, n_act_wg - 1) * ATT_SL, last = min(ATT_SL, end_wg - start) - 1;
#pragma unroll
            for (int n = 0; n < NU; ++n) {
                const int x = ht + 256 * n;
                const int r = x & 15, G8 = (x >> 4) % GQ, kt = (x >> 4) / GQ;
                const int j = min(pos_of(kt * 4 + (r & 3), r >> 2), last);
                const unsigned off = (unsigned)(start + j) * (HD * 2) + G8 * 64;   // (a KV head's plane is far below 4 GB)
#pragma unroll
                for (int w = 0; w < 4; ++w) kr[n][w] = *reinterpret_cast<const u32x4*>(kp + (off + w * 16));
                const int dq = x % DQ, uq = (x / DQ) & 3, gv = x / (DQ * 4);
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    vr[n][k] = *reinterpret_cast<const u32x2*>(vp + ((unsigned)(start + min(pos_of(uq * 8 + k, gv), last)) * (HD * 2) + dq * 8));
            }
        };
        auto stage = [&](int split) {
            const int start = min(split, n_act_wg - 1) * ATT_SL, npos = min(ATT_SL, end_wg - start);
#pragma unroll
            for (int n = 0; n < NU; ++n) {
                const int x = ht + 256 * n;
                // keys: fragment (key tile, 8 4-dim groups), lane (row r, gq)'s 16 bytes = dims 4 G + gq of those groups
                const int r = x & 15, G8 = (x >> 4) % GQ, kt = (x >> 4) / GQ;
                const bool ok = pos_of(kt * 4 + (r & 3), r >> 2) < npos;
                unsigned w[16];
#pragma unroll
                for (int e = 0; e < 4; ++e) { w[4 * e] = kr[n][e].x; w[4 * e + 1] = kr[n][e].y; w[4 * e + 2] = kr[n][e].z; w[4 * e + 3] = kr[n][e].w; }
#pragma unroll
                for (int gg = 0; gg < 4; ++gg) {
                    unsigned o[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        o[p] = pack_halves(w[4 * p + (gg >> 1)], w[4 * p + 2 + (gg >> 1)], gg & 1);
                        o[p] = ok ? o[p] : 0u;
                    }
                    *reinterpret_cast<u32x4*>(kb + ((kt * GQ + G8) * 64 + gg * 16 + r) * 16) = u32x4{o[0], o[1], o[2], o[3]};
                }
                // values: fragment (16-dim tile, 8 units), lane (dim r, gq)'s 16 bytes = those units' positions; the lanes'
                // places are XORed with the tile, or the 8 tiles a wave writes at once would share their banks
                const int dq = x % DQ, uq = (x / DQ) & 3, gv = x / (DQ * 4), dt = dq >> 2;
                u32x2 v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool vok = pos_of(uq * 8 + k, gv) < npos;
                    v[k] = u32x2{vok ? vr[n][k].x : 0u, vok ? vr[n][k].y : 0u};
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    unsigned o[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        o[p] = pack_halves((e >> 1) ? v[2 * p].y : v[2 * p].x, (e >> 1) ? v[2 * p + 1].y : v[2 * p + 1].x, e & 1);
                    const int place = (gv * 16 + (dq & 3) * 4 + e) ^ (dt & 7);
                    *reinterpret_cast<u32x4*>(vb + ((dt * 4 + uq) * 64 + place) * 16) = u32x4{o[0], o[1], o[2], o[3]};
                }
            }
        };

        fetch(sp);
        for (int s0 = 0; s0 < n_act_wg; s0 += 2) {
            const int split = s0 + sp;
            __syncthreads();                       // the previous pair (or merge) has been read
            stage(split);
            if (s0 + 2 < n_act_wg) fetch(split + 2);   // uniform over the workgroup
            __syncthreads();
            if (!live || split >= n_act) continue;     // uniform over the wave
            const int start = split * ATT_SL, npos = min(ATT_SL, end - start);

            // scores: unit u = kt * 4 + e of this lane's query in s[u].  The instructions of a block (8 4-dim groups of a key
            // tile) are issued with the tree of the previous block between them: both fit the 32 cycles an instruction
            // occupies the matrix core, and one wave alone keeps it busy.
            float s[32];
            {
                constexpr int NB = 8 * GQ;   // blocks
                auto key_frag = [&](int b) { return *reinterpret_cast<const u32x4*>(kb + (b * 64 + lane) * 16); };
                f32x4 d[2][8], part[GQ];
                u32x4 kf = key_frag(0);
#pragma unroll
                for (int b = 0; b <= NB; ++b) {
                    if (b < NB) {
                        const u32x4 kcur = kf;
                        if (b + 1 < NB) kf = key_frag(b + 1);
#pragma unroll
                        for (int G = 0; G < 8; ++G)
                            d[b & 1][G] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf16_of8(kcur, G), qv[(b % GQ) * 8 + G],
                                                                              f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    }
                    if (b > 0) {
                        f32x4* t = d[(b - 1) & 1];
#pragma unroll
                        for (int w = 1; w < 8; w <<= 1)
#pragma unroll
                            for (int i = 0; i + w < 8; i += 2 * w) t[i] = add4_rn(t[i], t[i + w]);
                        const int G8 = (b - 1) % GQ, kt = (b - 1) / GQ;
                        part[G8] = t[0];
                        if (G8 == GQ - 1) {
#pragma unroll
                            for (int w = 1; w < GQ; w <<= 1)
#pragma unroll
                                for (int i = 0; i + w < GQ; i += 2 * w) part[i] = add4_rn(part[i], part[i + w]);
                            const float pv[4] = {part[0].x, part[0].y, part[0].z, part[0].w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) s[kt * 4 + e] = mul_rn(pv[e], scale);
                        }
                    }
                    if (b < NB) {
#pragma unroll
                        for (int G = 0; G < 8; ++G) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a matrix-core instruction
                            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);   // and vector instructions under it
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const int n_seen = min(npos, my_pos - start + 1);   // positions of the split this lane's query attends to
            if (start + ATT_SL > a.pos0 + c * 16 + 1 || npos < ATT_SL) {   // uniform: the split reaches the tile's own rows
#pragma unroll
                for (int u = 0; u < 32; ++u) s[u] = pos_of(u, gq) < n_seen ? s[u] : -INFINITY;
            }
            // soft-max statistics: the maximum, and the sum in wave_sum's order (positions j and j + 64 first, then the
            // butterfly over 32, 16, .., 1: position bits are i, gq or the chain, highest bit first)
            float mx = s[0];
#pragma unroll
            for (int u = 1; u < 32; ++u) mx = fmaxf(mx, s[u]);
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
#pragma unroll
            for (int u = 0; u < 32; ++u) s[u] = mx > -INFINITY ? __expf(sub_rn(s[u], mx)) : 0.f;
            float R[NC / 4];   // R[x] of group gq: chain 4 x + gq, summed over its positions
#pragma unroll
            for (int x = 0; x < NC / 4; ++x) {
                float tt[4];
#pragma unroll
                for (int y = 0; y < 4; ++y) tt[y] = NI == 2 ? add_rn(s[(4 * x + y) * NI], s[(4 * x + y) * NI + NI - 1]) : s[4 * x + y];
                R[x] = fold16(fold32(tt[0], tt[2]), fold32(tt[1], tt[3]));
            }
#pragma unroll
            for (int w = NC / 8; w >= 1; w >>= 1)
#pragma unroll
                for (int x = 0; x < w; ++x) R[x] = add_rn(R[x], R[x + w]);
            float l = R[0];
            l = add_rn(l, __shfl_xor(l, 32));
            l = add_rn(l, __shfl_xor(l, 16));
            if (gq == 0)
                *reinterpret_cast<float2*>(slot_ml + ((size_t)split * PFX_QUERIES + tl * 16 + r16) * 2) = float2{mx, l};

            // values.  Rows past the tile's own chunk that another tile of the workgroup needed are zeros here, as in
            // attn_split (their probabilities are 0, but 0 times an infinity would not be)
            float* po = slot + ((size_t)split * PFX_QUERIES + tl * 16 + r16) * HD + gq * 4;
            auto values = [&](auto masked) {
#pragma unroll 2
                for (int dt = 0; dt < DT; ++dt) {
                    u32x4 vf[4];
#pragma unroll
                    for (int uq = 0; uq < 4; ++uq)
                        vf[uq] = *reinterpret_cast<const u32x4*>(vb + ((dt * 4 + uq) * 64 + (lane ^ (dt & 7))) * 16);
                    auto val = [&](int u) {
                        const float v = bf16_of8(vf[u >> 3], u & 7);
                        return masked.value && pos_of(u, gq) >= npos ? 0.f : v;
                    };
                    // four chains at a time, the previous four folded under them
                    constexpr int NG = NC / 4;
                    f32x4 tot = f32x4{0.f, 0.f, 0.f, 0.f}, o[2][4];
#pragma unroll
                    for (int q = 0; q <= NG; ++q) {
                        if (q < NG) {
#pragma unroll
                            for (int i = 0; i < NI; ++i)
#pragma unroll
                                for (int x = 0; x < 4; ++x) {
                                    const int u = (q * 4 + x) * NI + i;
                                    o[q & 1][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                        val(u), s[u], i == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : o[q & 1][x], 0, 0, 0);
                                }
                        }
                        if (q > 0) {
                            f32x4* t = o[(q - 1) & 1];
                            if constexpr (PPL == 2) {
                                tot = add4_rn(tot, add4_rn(t[0], t[1]));
                                tot = add4_rn(tot, add4_rn(t[2], t[3]));
                            } else {
                                static_assert(PPL == 2 || PPL == 4, "slots per wave");
                                tot = add4_rn(tot, add4_rn(add4_rn(t[0], t[1]), add4_rn(t[2], t[3])));
                            }
                        }
                        if (q < NG) {
#pragma unroll
                            for (int x = 0; x < 4 * NI; ++x) {
                                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    *reinterpret_cast<f32x4*>(po + dt * 16) = tot;
                }
            };
            if (npos < ATT_SL) values(std::true_type{}); else values(std::false_type{});
        }

        // merge: the splits' partials weighted by exp(max_s - max) in ascending split order, four outputs per thread.  The
        // statistics of as many queries as fit go to LDS first (none where one query's do not fit: a prompt of a million
        // positions and more; they are read where they lie then).
        const int fit = pf_mx_queries_in_lds((int)pfx_lds_bytes(HD), n_act_wg);
        const int qb = fit > 0 ? fit : PFX_QUERIES;
        for (int q0 = 0; q0 < PFX_QUERIES; q0 += qb) {
            const int nqb = min(qb, PFX_QUERIES - q0);
            float2* stat = reinterpret_cast<float2*>(lds);   // [n_act_wg][qb]
            __syncthreads();      // also: every wave's partials are written
            for (int e = tid; e < n_act_wg * nqb && fit > 0; e += WG_THREADS) {
                const int sI = e / nqb, ql = e - sI * nqb;
                stat[sI * qb + ql] = *reinterpret_cast<const float2*>(slot_ml + ((size_t)sI * PFX_QUERIES + q0 + ql) * 2);
            }
            __syncthreads();
            for (int e = tid; e < nqb * DQ; e += WG_THREADS) {
                const int ql = e / DQ, d0 = (e - ql * DQ) * 4, qi = q0 + ql, tq = tg * PFX_TILES + (qi >> 4);
                if (tq >= n_tk) continue;
                const int cq = tq / grp, m = cq * 16 + (qi & 15), hqq = g * grp + tq % grp;
                if (m >= a.M) continue;
                const int na = (chunk_end(cq) + ATT_SL - 1) / ATT_SL;
                auto ml_of = [&](int sI) {
                    return fit > 0 ? stat[sI * qb + ql] : *reinterpret_cast<const float2*>(slot_ml + ((size_t)sI * PFX_QUERIES + qi) * 2);
                };
                float gmax = -INFINITY;
                for (int sI = 0; sI < na; ++sI) gmax = fmaxf(gmax, ml_of(sI).x);
                const float* src = slot + (size_t)qi * HD + d0;
                float num[4] = {0.f, 0.f, 0.f, 0.f}, den = 0.f;
                for (int sb = 0; sb < na; sb += 8) {
                    f32x4 os[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        os[k] = *reinterpret_cast<const f32x4*>(src + (size_t)min(sb + k, na - 1) * (PFX_QUERIES * HD));
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        if (sb + k < na) {
                            const float2 ml = ml_of(sb + k);
                            const float w = (ml.x > -INFINITY) ? __expf(ml.x - gmax) : 0.f;
                            num[0] = fmaf(w, os[k].x, num[0]); num[1] = fmaf(w, os[k].y, num[1]);
                            num[2] = fmaf(w, os[k].z, num[2]); num[3] = fmaf(w, os[k].w, num[3]);
                            den = fmaf(w, ml.y, den);
                        }
                    }
                }
                *reinterpret_cast<f32x4*>(a.att + (size_t)m * H * HD + (size_t)hqq * HD + d0) =
                    f32x4{num[0] / den, num[1] / den, num[2] / den, num[3] / den};
            }
        }
        __syncthreads();   // the statistics have been read before the next item's keys overwrite them
    }
}

}  // namespace sdfp
