// Order of work on two streams of one call, whatever fails on the way.
#pragma once

namespace ff {

// First fork(), then first() (work on the caller's stream) and second() (on
// the other one), then join(): the caller's stream waits for the other one.
// Every step returns OK = Status() or an error.  Once the fork is done the
// join always runs, so that no error leaves work on the other stream that a
// later call on the caller's stream does not wait for; the error returned is
// the first one (second() does not run after first() failed).
template <class Fork, class First, class Second, class Join>
auto fork_join(const Fork& fork, const First& first, const Second& second, const Join& join) -> decltype(fork()) {
  using Status = decltype(fork());
  Status rc = fork();
  if (rc != Status()) return rc;
  rc = first();
  if (rc == Status()) rc = second();
  const Status rj = join();
  return rc != Status() ? rc : rj;
}

}  // namespace ff
