// Host-only logic of the library, free of any HIP call: the functor-chain
// compiler (Sec. 3.3, Tab. "functors"), the transfer-table bake, the camera
// basis and the screen rectangle of a job.  Compiled into the library and, on
// its own, into a sanitizer harness that feeds it hostile inputs on the CPU.
#pragma once

#include <string>

#include "isaac_internal.h"

namespace isaac {
namespace host {

struct CompiledChain {
    int n_ops = 0;
    int out_dim = 1;
    DevOp ops[kMaxOps];
};

// Parse "name(args) | name | ..." for an f_dim-component source into at most
// kMaxOps bytecode ops (after exact simplifications); false with a message in
// err on a bad chain.
bool compile_chain(const char* text, int f_dim, CompiledChain& out, std::string& err);

// T[j] = PL(j / 255), j = 0..255, as 4 floats per entry into table (256 x 4);
// false with a message on invalid points (fewer than 2, not spanning [0,1] with
// strictly increasing x, a value outside [0,1] or NaN).
bool bake_tf(const isaac_tf_point* pts, int n, float* table, std::string& err);

struct CameraBasis {
    double fwd[3], right[3], upp[3], h, aspect;
};

// Orthonormal forward/right/up' of a render descriptor's camera and the
// half-height of the view; false with a message for a degenerate camera.
bool camera_basis(const isaac_render_desc& j, CameraBasis& cb, std::string& err);

// A pixel rectangle [cull[0], cull[2]] x [cull[1], cull[3]] of the job's image
// containing every pixel whose ray can meet its box (from the job's camera,
// size, dims and origin); the whole image when a box corner lies at or behind
// the eye plane.
void set_cull_rect(DevJob& dj);

// What the rays of a launch are expected to be like.
struct RayLoad {
    double rays = 0.0;      // that meet their boxes
    double points = 0.0;    // scan points of each, to its end or its termination
    double spread = 0.0;    // pixels per voxel, times twice the step where that is more than one voxel:
                            // how much further apart a ray's own points lie than its neighbours'
    double pixels = 0.0;    // per voxel at the volume's centre
    double rows = 0.0;      // rows of voxels (y or z) between two scan points of a ray
};

// Lanes that evaluate a ray of the one-lane schedule: 1, or a group of 4 or 16 whose
// points are composited in order.  Every choice gives the same image.
int lanes_in_order(const RayLoad& l);

// Lanes per ray of iso-surface jobs whose schedule does not ask for 8 or more: 1 or 8,
// for the same image.
int lanes_iso(const RayLoad& l);

// Whether a trilinear point of a scalar whose x neighbours are adjacent takes its eight
// corners one by one rather than in pairs, where `lanes` lanes share a ray: the same image.
// clamp: at a border the corners are clamped (no guard layers).
bool corners_one_by_one(const RayLoad& l, int lanes, bool clamp);

}  // namespace host
}  // namespace isaac
