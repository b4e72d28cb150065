// A name that at most one process at a time holds: an abstract Unix socket bound to it, which the system gives back when the
// process ends, however it ends.  A forked child does not hold it (it closes its copy of the descriptor at once, or the name
// would stay taken for as long as the child lives).  The name space is the network name space's: processes in different ones
// (containers) do not see each other.
#pragma once
#include <pthread.h>
#include <sys/socket.h>
#include <sys/un.h>
#include <unistd.h>

#include <cerrno>
#include <cstddef>
#include <cstdio>
#include <cstring>

namespace sd {

class ProcessLock {
 public:
  // false: another process (or another lock of this one) holds the name, or it is not known whether one does
  bool take(const char* name) {
    static const int registered = pthread_atfork(nullptr, nullptr, close_all);
    if (registered != 0 || fd_ >= 0 || count_ >= kMost) return false;
    sockaddr_un address;
    const socklen_t n = named(address, name);
    if (n == 0) return false;
    const int fd = socket(AF_UNIX, SOCK_DGRAM | SOCK_CLOEXEC, 0);
    if (fd < 0) return false;
    if (bind(fd, reinterpret_cast<sockaddr*>(&address), n) != 0) {
      close(fd);
      return false;
    }
    fd_ = fd;
    held_[count_++] = this;
    return true;
  }
  // whether another lock holds that name, or it is not known that none does (asked through this one's socket: one that is not held does not know)
  bool held(const char* name) const {
    sockaddr_un address;
    const socklen_t n = named(address, name);
    return n == 0 || connect(fd_, reinterpret_cast<sockaddr*>(&address), n) == 0 || errno != ECONNREFUSED;
  }
  void drop() {
    if (fd_ < 0) return;
    close(fd_);
    fd_ = -1;
    for (int i = 0; i < count_; ++i)
      if (held_[i] == this) { held_[i] = held_[--count_]; break; }
  }

 private:
  // the name's address and its length (0: no such name)
  static socklen_t named(sockaddr_un& address, const char* name) {
    address = sockaddr_un{};
    address.sun_family = AF_UNIX;
    const int n = snprintf(address.sun_path + 1, sizeof address.sun_path - 1, "%s", name);
    return n < 1 || n >= (int)sizeof address.sun_path - 1 ? 0 : (socklen_t)(offsetof(sockaddr_un, sun_path) + 1 + n);
  }
  // (callers hold a mutex of their own around take and drop)
  static void close_all() {
    for (int i = 0; i < count_; ++i) { close(held_[i]->fd_); held_[i]->fd_ = -1; }
    count_ = 0;
  }
  static constexpr int kMost = 64;
  static inline ProcessLock* held_[kMost] = {};
  static inline int count_ = 0;
  int fd_ = -1;
};

}  // namespace sd
