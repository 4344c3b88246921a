// What the request queue needs to know about a pool (the pool itself stays opaque).
#pragma once
#include <hip/hip_runtime.h>
#include "../../include/hmi.h"

const hmi_pool_config_t* hmi_internal_config(const hmi_pool_t* pool);
hipStream_t hmi_internal_compute_stream(const hmi_pool_t* pool);
// every layer of the tenant has been registered (hmi_pool_load_tenant / hmi_pool_alias_tenant)
bool hmi_internal_tenant_ready(const hmi_pool_t* pool, int32_t tenant);
// whether a pool with a host tier has nothing on its compute stream: asked in front of work that belongs to the next forward call
bool hmi_internal_idle(hmi_pool_t* pool);
// hmi_stack_forward over all layers, told what hmi_internal_idle said in front of that work
int32_t hmi_internal_stack_forward(hmi_pool_t* pool, const void* x, void* y, const int32_t* tenant_ids, const int32_t* seq_lens, int32_t R,
                                   bool was_idle);
