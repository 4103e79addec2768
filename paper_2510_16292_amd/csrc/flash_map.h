// Which work item a workgroup of the prompt attention (flash.hip) takes.
// Plain C++, so that it can also be compiled for the host.
#pragma once
#ifdef __HIPCC__
#define QSVD_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define QSVD_HOST_DEVICE inline
#endif

namespace qsvd {

// Workgroup -> (group: a sequence's key/value head; wg: which of its n_wg
// workgroups).  The workgroups of one group read the same rows, so they get
// ids that one XCD receives (the chip hands workgroup i to XCD i % 8) and
// share its L2; the groups go round the XCDs one by one, so that sequences of
// different lengths spread over them, in `parts` interleaved parts each where
// that makes a multiple of eight.  Within an XCD, sets of so many parts as
// make about 128 workgroups (two rounds of its CUs) run one after the other,
// the workgroups with most keys of a set first.
constexpr int kFaSet = 128;

struct FaWork {
  int group, wg;
  bool any;        // false: nothing (the grid is rounded up)
};
QSVD_HOST_DEVICE FaWork fa_work(int block, int groups, int n_wg, int parts) {
  const int xcd = block & 7, slot = block >> 3;
  const int wpp = (n_wg + parts - 1) / parts;                   // workgroups per part
  const int ppx = (groups * parts + 7) / 8;                     // parts per XCD
  const int per_set = kFaSet / wpp > 1 ? kFaSet / wpp : 1;
  const int set = slot / (per_set * wpp), in_set = slot - set * per_set * wpp;
  const int left = ppx - set * per_set, n_in = left < per_set ? left : per_set;   // parts of this set
  const int part = xcd + 8 * (set * per_set + in_set % n_in);
  FaWork o;
  o.group = part / parts;
  o.wg = (wpp - 1 - in_set / n_in) * parts + part % parts;
  o.any = o.group < groups && o.wg < n_wg;
  return o;
}

inline int fa_parts(long long groups, int n_wg) {
  int parts = groups % 8 == 0 ? 1 : groups % 4 == 0 ? 2 : groups % 2 == 0 ? 4 : 8;
  while (parts > n_wg) parts /= 2;
  return parts;
}
inline long long fa_blocks(long long groups, int n_wg, int parts) {
  return (groups * parts + 7) / 8 * 8 * ((n_wg + parts - 1) / parts);
}

}  // namespace qsvd
