// Host check of csrc/process_lock.h, compiled and run by test_process_lock.py: prints the first condition that does not hold.
#include <sys/resource.h>
#include <sys/wait.h>

#include <cstdlib>

#include "../paper_2203_16487_amd/csrc/process_lock.h"

#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); exit(1); } } while (0)

// what another process gets for the name
static bool other_takes(const char* name) {
  const pid_t p = fork();
  if (p == 0) { sd::ProcessLock l; _exit(l.take(name) ? 1 : 0); }
  int status = 0;
  CHECK(waitpid(p, &status, 0) == p && WIFEXITED(status));
  return WEXITSTATUS(status) == 1;
}

int main(int, char** argv) {
  const char* name = argv[1];
  sd::ProcessLock a, b;
  CHECK(a.take(name));
  CHECK(!a.take(name));
  CHECK(!b.take(name));
  CHECK(!other_takes(name));
  a.drop();
  CHECK(other_takes(name));
  // a child forked while the name is held does not keep it from its parent
  CHECK(a.take(name));
  int go[2];
  CHECK(pipe(go) == 0);
  const pid_t child = fork();
  if (child == 0) { char c; close(go[1]); (void)!read(go[0], &c, 1); _exit(0); }
  a.drop();
  bool back = false;
  for (int i = 0; i < 1000 && !(back = a.take(name)); ++i) usleep(1000);   // (until the child has run)
  CHECK(back);
  close(go[1]);
  CHECK(waitpid(child, nullptr, 0) == child);
  a.drop();
  // asked, not taken: by a lock of another name, of this process and of others
  char second[256];
  snprintf(second, sizeof second, "%s-second", name);
  CHECK(a.held(name));          // (no socket of its own to ask through)
  CHECK(a.take(second));
  CHECK(!a.held(name));
  CHECK(b.take(name));
  for (int i = 0; i < 3; ++i) CHECK(a.held(name));
  CHECK(!other_takes(name));
  b.drop();
  CHECK(!a.held(name));         // (having asked does not keep it)
  CHECK(other_takes(name));
  int up[2], down[2];
  CHECK(pipe(up) == 0 && pipe(down) == 0);
  const pid_t holder = fork();
  if (holder == 0) {
    sd::ProcessLock l;
    char c = l.take(name) ? 'y' : 'n';
    (void)!write(up[1], &c, 1);
    close(down[1]);
    (void)!read(down[0], &c, 1);
    _exit(0);
  }
  char c = 0;
  CHECK(read(up[0], &c, 1) == 1 && c == 'y');
  CHECK(a.held(name));
  close(down[1]);
  CHECK(waitpid(holder, nullptr, 0) == holder);
  CHECK(!a.held(name));         // (gone with its process)
  a.drop();
  // no socket to be had, or no such name: not the holder
  char longer[256];
  memset(longer, 'x', sizeof longer - 1);
  longer[sizeof longer - 1] = 0;
  CHECK(!a.take(longer));
  rlimit none{0, 0};
  CHECK(setrlimit(RLIMIT_NOFILE, &none) == 0);
  CHECK(!a.take(name));
  return 0;
}
