// The types of the HIP runtime that librasp's host-side headers name, for tests
// of those headers on the CPU.
#pragma once
#include <stdint.h>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
struct Stream;
typedef Stream *hipStream_t;
