#pragma once
#include "hip_runtime.h"
typedef _Float16 __half;
inline uint16_t __half_as_ushort(__half h) {
    uint16_t u;
    memcpy(&u, &h, 2);
    return u;
}
