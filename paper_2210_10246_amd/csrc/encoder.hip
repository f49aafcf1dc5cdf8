// The launches of encoder.h.  Heads are taken from and put into the [T, 3 hidden] and [T, hidden] layouts by the
// strides of the products, and residuals, biases, 1 / sqrt(d) and the sums for the bias gradients are part of them: no
// copies, no elementwise passes beside the three layers; GELU is part of the products around it.
#include <algorithm>
#include <cmath>

#include "encoder.h"
#include "matmul.h"

namespace tempo {
namespace {

struct Sizes {
  int64_t T, H, F, S, d;
  int B, A;
  explicit Sizes(const tempo_encoder& e)
      : T(e.batch * e.seq), H(e.hidden), F(e.ffn), S(e.seq), d(e.hidden / e.heads), B(static_cast<int>(e.batch)),
        A(static_cast<int>(e.heads)) {}
};

MatSide rows_of(const float* p, int64_t ld, int64_t outer = 0, int64_t inner = 0) { return {p, ld, outer, inner, false}; }
MatSide columns_of(const float* p, int64_t ld, int64_t outer = 0, int64_t inner = 0) { return {p, ld, outer, inner, true}; }

Matmul product(MatSide a, MatSide b, float* c, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  return {a, b, c, ldc, 0, 0, nullptr, nullptr, nullptr, 1.0f, static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), 1, 1,
          static_cast<int>(N)};
}
// One product per head.
Matmul per_head(const Sizes& z, MatSide a, MatSide b, float* c, int64_t ldc, int64_t c_outer, int64_t c_inner, int64_t N,
                int64_t K) {
  Matmul g = product(a, b, c, ldc, z.S, N, K);
  g.c_outer = c_outer;
  g.c_inner = c_inner;
  g.batch = z.B * z.A;
  g.inner = z.A;
  return g;
}
// y = x w^T + bias (+ add)
Matmul linear(const float* x, const float* w, const float* bias, const float* add, float* y, int64_t T, int64_t out, int64_t in) {
  Matmul g = product(rows_of(x, in), rows_of(w, in), y, out, T, out, in);
  g.bias = bias;
  g.add = add;
  return g;
}
// dx = dy w (+ add)
Matmul linear_dx(const float* dy, const float* w, const float* add, float* dx, int64_t T, int64_t out, int64_t in) {
  Matmul g = product(rows_of(dy, out), columns_of(w, in), dx, in, T, in, out);
  g.add = add;
  return g;
}
// dw = dy^T x and db = the column sums of dy, either of which may be null.  Where only db is wanted, x need not be there: the
// tiles that make the sums take dy for it, and nothing stores what they multiply.
Matmul linear_dw(const float* dy, const float* x, float* dw, float* db, int64_t T, int64_t out, int64_t in) {
  Matmul g = product(columns_of(dy, out), dw ? columns_of(x, in) : columns_of(dy, out), dw, in, out, dw ? in : std::min(in, out), T);
  g.n_counted = static_cast<int>(in);
  g.a_sums = db;
  return g;
}

// The layer's GELU at the end of a product: the forward's of the first feed-forward layer, the backward's of the second one's
// dx.  As launches of their own they took 4.5 us each at 2 x 128 x 768 and read and wrote [T, ffn] once more: a replayed step
// 203.5 / 197.8 us, 8 x 256 x 768 1019 / 998.  The mask is bytes to the product: rows of a multiple of 8 columns.
void with_gelu(Matmul& g, const tempo_encoder& e, Matmul::Act act) {
  g.act = act;
  g.kind = e.kind;
  g.act_y = e.h;
  g.side = reinterpret_cast<uint8_t*>(e.side);
}

struct Run {
  hipStream_t st;
  tempo_status status = TEMPO_OK;
  void operator()(tempo_status s) {
    if (status == TEMPO_OK) status = s;
  }
  void operator()(const Matmul& g) {
    if (status == TEMPO_OK) status = launch_matmul(g, st);
  }
  // A layer's dx, and its dw and db, any of which may not be wanted.
  void backward(const Matmul& dx, const Matmul& dw) {
    if (status == TEMPO_OK && (dx.c || dw.c || dw.a_sums)) status = launch_matmul_group(dx, dw, nullptr, st);
  }
};

}  // namespace
}  // namespace tempo

using namespace tempo;

int tempo_encoder_takes(const tempo_encoder* e) {
  const int64_t most = int64_t{1} << 30;
  for (int64_t n : {e->batch, e->seq, e->hidden, e->heads, e->ffn})
    if (n < 1 || n > most) return 0;
  if (e->hidden % e->heads != 0) return 0;
  const Sizes z(*e);
  if (z.H % 4 != 0 || z.F % 4 != 0 || z.d % 4 != 0) return 0;
  // Elements of every tensor; then tiles: sizes, tiles and lanes are counted in 32 bits, and a launch has up to three products
  // of 256 lanes a tile, at least 32 x 32 elements each.
  const int64_t slices = e->batch * e->heads;
  if (z.T > most / (3 * z.H) || z.T > most / z.F || z.F > most / z.H || z.S > 32768 || slices > most / (z.S * z.S)) return 0;
  auto tiles = [](int64_t M, int64_t N) { return (M + kTile - 1) / kTile * ((N + kTile - 1) / kTile); };
  for (int64_t n : {tiles(z.T, 3 * z.H), tiles(z.T, z.F), tiles(3 * z.H, z.H), tiles(z.F, z.H), slices * tiles(z.S, z.S),
                    slices * tiles(z.S, z.d)})
    if (n > most / (kTile * kTile)) return 0;
  // Where the launches, copies and host time that go count for more than the library's products gain.  us of the parts / of this,
  // forward + backward and, behind a comma, forward alone, of four runs in turn the fastest.
  // Rows of attention: longer ones leave both to the attention kernels and the library's products win.  1 x 6144 x 256 in 4 heads
  // 3967 / 3655, 1528 / 1393, 1 x 7168 x 256 5383 / 4904, 2086 / 1832; 1 x 8192 x 256 6440 / 6442, 2569 / 2498, 1 x 8192 x 128 in 2
  // 3388 / 3452, 1320 / 1309, 1 x 16384 x 64 in 1 6466 / 6712, 2500 / 2493.
  if (z.S > 7168) return 0;
  // Multiplications of the four layers' weights, forward: 2 x 128 x 768 (2e9) 814 / 197, 243 / 76, 8 x 128 x 1024 (13e9) 950 / 775,
  // 310 / 274, 14 x 256 x 768 (25e9) 1863 / 1629, 613 / 534, 8 x 256 x 1024 (26e9) 1570 / 1469, 518 / 497, 32 x 256 x 512 (26e9) 1820
  // / 1774, 594 / 575.  Beyond, it is 2 to 8 % one way or the other from run to run: 10 x 256 x 1024 (32e9) 1970 / 1904, 655 / 647, 12
  // x 256 x 1024 (39e9) 2239 / 2164 (another day 2269 / 2326), 24 x 256 x 768 (43e9) 2908 / 2833, 48 x 256 x 512 (39e9) 2714 / 2649
  // (2742 / 2776), 64 x 256 x 512 (52e9) 3439 / 3549, 16 x 256 x 1024 (52e9) 2890 / 3095.
  const int64_t weights = 4 * z.H * z.H + 2 * z.H * z.F, products = z.T * weights, billion = 1000 * 1000 * 1000;
  if (weights <= 30 * 1000 * 1000 && z.d <= 256) return products <= 26 * billion;
  // Layers wider than 1536 columns: rows count in whole tiles, and the weights themselves count (as 47 more rows; the library streams
  // them faster).  Heads wider than 256: their own products are as large (counted twice, as there are two each way; the library's are
  // faster).  256 x 2048 1044 / 798, 313 / 267, 190 x 2304 1160 / 812, 312 / 290, 60 x 3072 1043 / 633, 230 / 210, 8 x 4096 1077 / 771,
  // 248 / 231; at its worst 100 x 2560 929 / 717, 253 / 274, 24 x 4096 991 / 813, 228 / 237; not taken 257 x 2048 1031 / 952, 311 / 331,
  // 500 x 2048 1481 / 1442, 456 / 500, 81 x 3072 1012 / 874, 287 / 317, 80 x 4096 1310 / 1345, 402 / 451, 1 x 5120 1127 / 1084, 302 /
  // 312, 1 x 8192 2029 / 3561, 586 / 606, 8 x 12288 4448 / 6951, 1332 / 1426.  In one head: 1900 x 512 1033 / 694, 230 / 228; not taken
  // 4096 x 512 1687 / 1732, 545 / 579, 1024 x 1024 993 / 836, 273 / 295, 2048 x 1024 1732 / 1799, 558 / 603.
  const int64_t rows = (z.T + kTile - 1) / kTile * kTile + 47, attention = z.d > 256 ? 2 * 2 * z.T * z.S * z.H : 0;
  return rows * weights + attention <= 16 * billion;
}

tempo_status tempo_encoder_fwd(const tempo_encoder* e, float* out, void* hip_stream) {
  const Sizes z(*e);
  const int64_t H = z.H, S = z.S, d = z.d, L = 3 * H;
  const float scale = static_cast<float>(1.0 / std::sqrt(static_cast<double>(d)));
  Run run{static_cast<hipStream_t>(hip_stream)};
  run(linear(e->x, e->wqkv, e->bqkv, nullptr, e->qkv, z.T, L, H));
  Matmul scores = per_head(z, rows_of(e->qkv, L, S * L, d), rows_of(e->qkv + H, L, S * L, d), e->probs, S, z.A * S * S, S * S, S, d);
  scores.alpha = scale;
  run(scores);
  if (run.status == TEMPO_OK)
    run(tempo_attn_softmax_dropout_fwd(e->probs, e->key_len, 0, e->probs, out, e->keep, e->batch, e->heads, S, S, e->p,
                                       e->seed, e->offset, TEMPO_F32, hip_stream));
  run(per_head(z, rows_of(out, S, z.A * S * S, S * S), columns_of(e->qkv + 2 * H, L, S * L, d), e->ctxt, H, S * H, d, d, S));
  run(linear(e->ctxt, e->wproj, e->bproj, e->x, e->y1, z.T, H, H));
  if (run.status == TEMPO_OK)
    run(tempo_layernorm_fwd(e->y1, e->gamma1, e->beta1, e->y1, e->rstd1, nullptr, z.T, H, e->eps1, TEMPO_F32, hip_stream));
  Matmul h = linear(e->y1, e->w1, e->b1, nullptr, e->h, z.T, z.F, H);
  if (z.F % 8 == 0) with_gelu(h, *e, Matmul::kForward);
  run(h);
  if (z.F % 8 != 0 && run.status == TEMPO_OK)
    run(tempo_gelu_fwd(e->h, e->h, e->side, z.T * z.F, TEMPO_F32, e->kind, hip_stream));
  run(linear(e->h, e->w2, e->b2, e->y1, e->y2, z.T, H, z.F));
  if (run.status == TEMPO_OK)
    run(tempo_layernorm_fwd(e->y2, e->gamma2, e->beta2, e->y2, e->rstd2, nullptr, z.T, H, e->eps2, TEMPO_F32, hip_stream));
  return run.status;
}

tempo_status tempo_encoder_bwd_ffn(const tempo_encoder* e, const tempo_encoder_grads* g, const float* dy, float* ds2,
                                   float* dh, float* dy1, void* workspace, size_t workspace_bytes, void* hip_stream) {
  const Sizes z(*e);
  Run run{static_cast<hipStream_t>(hip_stream)};
  run(tempo_layernorm_bwd(dy, e->y2, e->gamma2, e->beta2, e->rstd2, ds2, g->dgamma2, g->dbeta2, workspace, workspace_bytes,
                          z.T, z.H, TEMPO_F32, hip_stream));
  const bool more = dy1 || g->dw1 || g->db1;
  Matmul dh2 = linear_dx(ds2, e->w2, nullptr, more ? dh : nullptr, z.T, z.H, z.F);
  if (z.F % 8 == 0) with_gelu(dh2, *e, Matmul::kBackward);
  run.backward(dh2, linear_dw(ds2, e->h, g->dw2, g->db2, z.T, z.H, z.F));
  if (!more) return run.status;
  if (z.F % 8 != 0 && run.status == TEMPO_OK) run(tempo_gelu_bwd(dh, e->h, e->side, dh, z.T * z.F, TEMPO_F32, e->kind, hip_stream));
  run.backward(linear_dx(dh, e->w1, ds2, dy1, z.T, z.F, z.H), linear_dw(dh, e->y1, g->dw1, g->db1, z.T, z.F, z.H));
  return run.status;
}

tempo_status tempo_encoder_bwd_norm(const tempo_encoder* e, const tempo_encoder_grads* g, const float* dy1, float* ds1,
                                    void* workspace, size_t workspace_bytes, void* hip_stream) {
  const Sizes z(*e);
  return tempo_layernorm_bwd(dy1, e->y1, e->gamma1, e->beta1, e->rstd1, ds1, g->dgamma1, g->dbeta1, workspace,
                             workspace_bytes, z.T, z.H, TEMPO_F32, hip_stream);
}

tempo_status tempo_encoder_bwd_attention(const tempo_encoder* e, const tempo_encoder_grads* g, const float* ds1,
                                         float* dctxt, float* dqkv, float* dout, float* out, void* hip_stream) {
  const Sizes z(*e);
  const int64_t H = z.H, S = z.S, d = z.d, L = 3 * H, SS = S * S;
  const float scale = static_cast<float>(1.0 / std::sqrt(static_cast<double>(d)));
  Run run{static_cast<hipStream_t>(hip_stream)};
  run.backward(linear_dx(ds1, e->wproj, nullptr, dctxt, z.T, H, H), linear_dw(ds1, e->ctxt, g->dwproj, g->dbproj, z.T, H, H));
  if (!dctxt) return run.status;
  run(per_head(z, rows_of(dctxt, H, S * H, d), rows_of(e->qkv + 2 * H, L, S * L, d), dout, S, z.A * SS, SS, S, d));
  if (run.status == TEMPO_OK) {
    if (e->keep)
      run(tempo_attn_softmax_dropout_bwd(dout, e->probs, e->keep, dout, out, e->batch, e->heads, S, S, e->p, TEMPO_F32, hip_stream));
    else
      run(tempo_attn_softmax_dropout_bwd_regen(dout, e->probs, dout, out, e->batch, e->heads, S, S, e->p, e->seed,
                                               e->offset, TEMPO_F32, hip_stream));
  }
  const Matmul dv = per_head(z, columns_of(out, S, z.A * SS, SS), columns_of(dctxt, H, S * H, d), dqkv + 2 * H, L, S * L, d, d, S);
  Matmul dq = per_head(z, rows_of(dout, S, z.A * SS, SS), columns_of(e->qkv + H, L, S * L, d), dqkv, L, S * L, d, d, S);
  Matmul dk = per_head(z, columns_of(dout, S, z.A * SS, SS), columns_of(e->qkv, L, S * L, d), dqkv + H, L, S * L, d, d, S);
  dq.alpha = dk.alpha = scale;
  if (run.status == TEMPO_OK) run(launch_matmul_group(dq, dk, &dv, run.st));
  run.backward(linear_dx(dqkv, e->wqkv, ds1, g->dx, z.T, L, H), linear_dw(dqkv, e->x, g->dwqkv, g->dbqkv, z.T, L, H));
  return run.status;
}
