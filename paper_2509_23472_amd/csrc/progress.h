// What a solving workgroup of the fused factor-and-solve launch makes of the progress word (ortho_f64.h).  Plain C++, so
// that the rules can be tested without a GPU.
#pragma once

#ifdef __HIPCC__
#define CF_FN __host__ __device__ __forceinline__
#else
#define CF_FN inline
#endif

// Progress word: (attempt << 16) | panels, where `panels` = p means that block columns 0 .. p-1 of L and the inverted
// diagonal blocks 0 .. p-1 are complete in memory, and `attempt` counts restarts of the factorisation (what a
// solving workgroup consumed of an abandoned attempt is worthless, so it starts over).  Within a launch the word only
// ever grows: a smaller one than was seen before is a poll that was sent off earlier.
#define CF_ATTEMPT_SHIFT 16
CF_FN constexpr int cf_word(int attempt, int panels) { return (attempt << CF_ATTEMPT_SHIFT) | panels; }

// A solving workgroup's place in the factorisation.
struct CfProgress {
  int attempt = 0;
  int known = 0;            // the largest word seen
};
enum { CF_TAKE, CF_RESTART, CF_GIVE_UP };

// Waits until there is something to do about panel J: CF_TAKE, it is complete; CF_RESTART, its attempt was abandoned, and
// p.attempt is the one to start over with; CF_GIVE_UP, neither after `limit` polls.  poll(spin) is the word of poll `spin`,
// the same for every thread of the workgroup; poll(0) may be older than words that were seen already.
template <class Poll>
CF_FN int cf_wait_panel(CfProgress& p, int J, int limit, Poll poll) {
  const int before = cf_word(p.attempt, J);      // words up to this one: not complete (or an earlier attempt's)
  for (int spin = 0; p.known <= before; ++spin) {
    if (spin == limit) return CF_GIVE_UP;
    const int f = poll(spin);
    if (f > p.known) p.known = f;
  }
  if ((p.known >> CF_ATTEMPT_SHIFT) == p.attempt) return CF_TAKE;
  p.attempt = p.known >> CF_ATTEMPT_SHIFT;
  return CF_RESTART;
}
