// Stand-ins for the library's entry points behind the binding's native code:
// each counts its call; the slow one takes a second, as a call that waits.
#include <unistd.h>

int stub_calls = 0;

int stub_call(void) {
  ++stub_calls;
  return 0;
}

int stub_slow_call(void) {
  usleep(1000000);
  return 0;
}
