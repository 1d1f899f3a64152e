// Host check of the passes of calls of more than 64 tokens: whatever the call, the regions of every
// pass that is launched lie inside the workspace that ffn_workspace_bytes asks for, and the row chunks
// of the down grid fit its workgroups' lists; likewise the regions of a pass of 33..64 tokens.
// Prints "calls passes" and exits 0, or the first pass that does not fit and exits 1.
#include <cstdio>
#include <cstdint>

#include "ffn_internal.h"

namespace {

int64_t g_calls = 0, g_passes = 0;

bool check(int wdt, int T, int d, int d_ff, int r, bool has_g, size_t extra) {
  static const int32_t idx = 0;
  ffn::Form form;
  if (has_g) form.g_idx = &idx;  // never read here
  const ffn::Gate g = r > 0 ? ffn::Gate::LoPA : ffn::Gate::Standard;
  char* const base = reinterpret_cast<char*>(uintptr_t(1) << 20);  // never dereferenced
  ffn::Workspace ws;
  const size_t need = ffn::workspace_layout(T, d, d_ff, r, base, &ws), bytes = need + extra;
  const size_t head = ffn::pass_head(ws, base);
  const int wide = ffn::wide_pass_tokens(ffn::Shape{T, d, d_ff, r, wdt, {}}, g, form, head, bytes);
  const int per = wide > 0 ? wide : ffn::kTokChunk;
  ++g_calls;
  if (wide != 0 && (wide <= ffn::kTokChunk || wide > ffn::kWidePass || wide % 16 != 0)) {
    std::printf("passes of %d tokens: T %d d %d d_ff %d r %d\n", wide, T, d, d_ff, r);
    return false;
  }
  for (int t0 = 0; t0 < T; t0 += per) {
    const ffn::Shape pass{T - t0 < per ? T - t0 : per, d, d_ff, r, wdt, {}};
    if (pass.T <= ffn::kTokChunk) continue;
    ++g_passes;
    const size_t used = ffn::wide_pass_bytes(pass, g, form, head);
    if (used > bytes) {
      std::printf("pass of %d tokens uses %zu of %zu bytes: T %d d %d d_ff %d r %d G %d weights %d\n", pass.T, used, bytes, T,
                  d, d_ff, r, has_g, wdt);
      return false;
    }
  }
  return true;
}

// The row chunks of the down grid fit its workgroups' lists.
bool check_chunks(int units, int d_ff, int nseg) {
  const int R = ffn::wide_down_chunks(units, d_ff, nseg);
  const int rows = (d_ff + nseg - 1) / nseg, segs = R > 0 ? (nseg + R - 1) / R : 0;
  if (R >= 1 && R <= nseg && segs <= ffn::kWDnSegs && segs * rows <= ffn::kWDnRows) return true;
  std::printf("%d chunks: %d units, d_ff %d, %d segments\n", R, units, d_ff, nseg);
  return false;
}

// A pass of 33..64 tokens on the wide kernels uses the workspace's own regions: z's first copy and zval
// lie in zf, z's planes in seg_zval.  `taken` counts the calls that the path takes.
bool check_64(int wdt, int T, int tc, int d, int d_ff, int r, int64_t* taken) {
  ffn::Workspace ws;
  ffn::workspace_layout(tc, d, d_ff, r, reinterpret_cast<char*>(uintptr_t(1) << 20), &ws);
  if (!ffn::wide64_ok(ffn::Shape{T, d, d_ff, r, wdt, {}}, r > 0 ? ffn::Gate::LoPA : ffn::Gate::Standard, ws)) return true;
  ++*taken;
  const int64_t ntt = (tc + 15) / 16, nseg = (d_ff + 63) / 64;
  const int64_t zf = reinterpret_cast<char*>(ws.xs) - reinterpret_cast<char*>(ws.zf);
  const int64_t zval = reinterpret_cast<char*>(ws.z) - reinterpret_cast<char*>(ws.seg_zval);
  if (T >= ffn::kWide64Min && tc <= ffn::kTokChunk && 16 * 16 * 16 * ntt * nseg <= zf && 4 * (int64_t)T * r <= zf &&
      16 * 2 * 64 * ((r + 31) / 32) * ntt <= zval)
    return true;
  std::printf("33..64 tokens do not fit: T %d of %d, d %d, d_ff %d, r %d, weights %d\n", T, tc, d, d_ff, r, wdt);
  return false;
}

uint64_t g_state = 88172645463325252ull;
uint32_t next(uint32_t n) {  // 0 .. n - 1
  g_state ^= g_state << 13, g_state ^= g_state >> 7, g_state ^= g_state << 17;
  return (uint32_t)((g_state >> 16) % n);
}

}  // namespace

int main() {
  // calls whose smaller passes need more workspace than a larger one: 256-token and 128-token
  // passes with a rank near d_ff / 2
  const int known[][5] = {{128, 6656, 13189, 6656, 1}, {128, 2728, 17675, 8872, 1}, {256, 2280, 9111, 4592, 0},
                          {508, 2112, 9510, 4792, 0},  {486, 5464, 15401, 7720, 1}};
  for (const auto& k : known)
    if (!check(1, k[0], k[1], k[2], k[3], k[4] != 0, 0)) return 1;
  for (int i = 0; i < 20000; ++i) {
    const int d_ff = 1 + (int)next(next(2) ? 1 << 20 : 30000), rows = next(2) ? 64 : 128;
    if (!check_chunks(1 + (int)next(300), d_ff, (d_ff + rows - 1) / rows)) return 1;
  }
  int64_t taken = 0;
  for (int i = 0; i < 100000; ++i) {
    const int wdt = 1 + (int)next(3), q = wdt == 1 ? 8 : wdt == 2 ? 16 : 32;
    const int T = 2 + (int)next(63), tc = next(2) ? T : 64, d_ff = 1 + (int)next(40000);
    const int r = next(3) ? (int)((next(2) ? d_ff + next(400) : next(2 * d_ff)) / q * q) : 0;
    if (!check_64(wdt, T, tc, q * (1 + (int)next(8192 / q)), d_ff, r, &taken)) return 1;
  }
  if (taken < 1000) return 1;
  for (int i = 0; i < 400000; ++i) {
    const int wdt = 1 + (int)next(3), q = wdt == 1 ? 8 : wdt == 2 ? 16 : 32;
    const int d = q * (1 + (int)next(8192 / q)), d_ff = 1 + (int)next(next(2) ? 30000 : 2000);
    int r = 0;
    if (next(4) != 0) {
      // over all ranks, and around half of d_ff, where z's copies stop fitting in zval's space
      const int near = d_ff / 2 + (int)next(401) - 200;
      const int v = next(2) ? (near > 0 ? near : 1) : 1 + (int)next(d_ff);
      r = (v + q - 1) / q * q;
    }
    const int T = 65 + (int)next(next(2) ? 1936 : 250);
    if (!check(wdt, T, d, d_ff, r, r > 0 && next(2) != 0, next(3) ? 0 : (size_t)next(1 << 24))) return 1;
  }
  std::printf("%lld %lld\n", (long long)g_calls, (long long)g_passes);
  return 0;
}
