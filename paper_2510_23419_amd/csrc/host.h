// host.h — host-only helpers of libpbit (no HIP types): error reporting, the
// FP64 minority-threshold table and the greedy colouring.
#pragma once

#include <stdint.h>

#include <string>

namespace pbit {

int fail(int code, const char *fmt, ...);
// Puts the thread's error message back at the end of its scope: around an attempt that the call
// can do without.
class KeepError {
public:
    KeepError();
    ~KeepError();
    KeepError(const KeepError &) = delete;
    KeepError &operator=(const KeepError &) = delete;

private:
    std::string saved;
};
uint32_t minority_threshold(double beta, int a);
int table_width(const double *beta, int S, int amax);
void build_table(const double *beta, int S, int width, uint32_t *out, int max_threads = 16);
int greedy_colouring(int n, int n_bonds, const int32_t *bi, const int32_t *bj, uint8_t *colour, int *n_colours);

}  // namespace pbit
