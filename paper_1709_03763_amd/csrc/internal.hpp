// Host-side helpers shared between the translation units of libscsurf.
#pragma once

#include "common.hpp"

namespace sc {

// Device scratch (see scratch.cpp): `p` null when there is no memory.  `idle`:
// the device has finished with the buffer; else it is freed, which waits.
struct Scratch {
    unsigned char* p = nullptr;
    size_t bytes = 0;
    int device = 0;
};
Scratch scratch_take(size_t bytes);
void scratch_give(Scratch& s, bool idle);
void scratch_trim();
// A volume begins (+1) or ends (-1).
void scratch_volumes(int change);

// hipMalloc; where there is no memory, once more without the kept scratch.
// Leaves no error behind.
bool device_alloc_bytes(void** p, size_t bytes);
template <class T>
bool device_alloc(T** p, size_t bytes)
{
    return device_alloc_bytes(reinterpret_cast<void**>(p), bytes);
}

// Parts of one buffer, 256-byte aligned.
struct Carve {
    unsigned char* base;
    size_t off = 0;
    template <class T>
    T* take(size_t n)
    {
        T* t = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off = (off + sizeof(T) * n + 255) & ~size_t(255);
        return t;
    }
};

void fill_u64(uint64_t* p, uint64_t v, size_t n, hipStream_t s);
void fill_u32(uint32_t* p, uint32_t v, size_t n, hipStream_t s);
void make_op(const sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T, int sign,
             int kf_index, OpDesc* op);
bool keyframe_ok(const sc_keyframe* kf);
OpDesc* stage_begin(sc_volume* vol);
BatchHdr* stage_hdr(sc_volume* vol);
sc_status stage_end(sc_volume* vol, hipStream_t s);
int cand_batch_resident_wgs(int variant);
sc_status run_candidates(sc_volume* vol, const OpDesc* ops, int n_ops, const sc_intrinsics* in, hipStream_t s);
void rec_clear(sc_volume* vol);
void rec_destroy(sc_volume* vol);
void rec_for_integration(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T,
                         bool records, OpDesc* op);
void rec_for_deintegration(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T,
                           OpDesc* op);
void rec_commit(sc_volume* vol);
sc_status stream_in_batch(sc_volume* vol, hipStream_t s);
sc_status stream_in_plain(sc_volume* vol, int parity, hipStream_t s);
void stream_clear(sc_volume* vol);
void stream_destroy(sc_volume* vol);
int64_t stream_host_blocks(const sc_volume* vol);
sc_status plain_op(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T, int sign,
                   hipStream_t s);

}  // namespace sc
