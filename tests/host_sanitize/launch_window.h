// What the driver and the stand-ins of the kernel launchers share: the workspace that the caller of
// the running iteration brought, and how many layers of each kind of work were launched.
#pragma once
#include <cstddef>

struct LaunchWindow {
    bool open;
    const void* workspace;
    size_t bytes;
    int layers_appended, layers_decoded, layers_prefilled;
};
extern LaunchWindow g_window;
