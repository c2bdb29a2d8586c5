// The streamer needs nothing of the device code on the host.
#pragma once
#include "graph.hpp"
