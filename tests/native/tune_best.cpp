// Feeds trial times to the tuner's comparison: "c <candidate> <ms>" to the on-chip
// form's best, "s <candidate> <ms>" to the streaming form's. Prints both and which
// form is taken.
#include <cstdio>
#include <cstdlib>

#include "sos_tune.h"

int main(int argc, char** argv) {
  sos::TuneBest chip, stream;
  for (int i = 1; i + 2 < argc; i += 3)
    (argv[i][0] == 'c' ? chip : stream).offer(atoi(argv[i + 1]), atof(argv[i + 2]));
  printf("%d %.6f %d %.6f %s\n", chip.which, chip.ms, stream.which, stream.ms,
         sos::tune_replaces(stream, chip) ? "streaming" : "chip");
  return 0;
}
