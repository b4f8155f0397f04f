// The programs here hold host code only: nothing is registered with the HIP
// runtime at start-up (there is no device code to register).
#pragma once
#include <cstddef>

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* none = nullptr;
  return &none;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*,
                           void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}
