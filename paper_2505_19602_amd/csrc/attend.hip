// Unmasked attention of the current token map over [retained cache ; current
// map] (Sec. 3.1 / 3.3): out[t] = sum_i softmax_i(q_t . k_i * sm_scale) v_i.
// Which kernel takes which shape: attend_f32.hip everything in fp32, step_small.hip bf16 where
// small_tile_rows() says so, attend_pipe.hip the rest.
#include "common.h"

namespace scalekv {

hipError_t launch_attend(int dtype, int n_seq, int n_head, int d, const void* q, int n_q, KvView k,
                         KvView v, int kv_len, float sm_scale, void* out, hipStream_t stream) {
  const int n_unit = n_seq * n_head;
  if (n_q <= 0 || n_unit <= 0) return hipSuccess;
  if (dtype == 0)
    return launch_attend_f32(n_unit, n_head, d, q, n_q, k, v, kv_len, sm_scale, out, stream);
  const int rows = small_tile_rows(dtype, d, n_unit, n_q, kv_len, SmallWork::kAttend);
  if (rows == 0)
    return launch_attend_pipe(n_unit, n_head, d, q, n_q, k, v, kv_len, nullptr, nullptr, 0, nullptr, sm_scale, out,
                              stream);
  SmallStep s{};
  s.n_unit = n_unit; s.n_head = n_head; s.d = d;
  s.q = q; s.n_q = n_q; s.tile_rows = rows; s.out = out;
  s.k = k; s.v = v; s.len1 = kv_len;
  s.sm_scale = sm_scale;
  return launch_step_small(s, stream);
}

}  // namespace scalekv
